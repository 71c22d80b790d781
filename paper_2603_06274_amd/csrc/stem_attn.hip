// Stage 3 (Algorithm 1 step 3d): block-sparse causal flash attention over the selected key blocks.
//
// One workgroup owns one (query head, query block): B query rows, 32 (or 16) per wavefront.  Per listed key
// block each wave runs
//     S^T = K Q^T      A = K rows from LDS, B = the wave's Q rows (registers)
//     online softmax   exp2 domain, fp32
//     O^T += V^T P^T   A = V^T rows read from row-major V in LDS with ds_read_b64_tr_b16,
//                      B = P^T taken straight from the S^T accumulators
// Computing the transposed products puts one query in one lane (and its partners at the same lane number modulo 16),
// so the softmax row reductions are in-lane plus an exchange between those lanes, and the S^T accumulator
// registers are already in the B-operand layout of the second product.
//
// K and V blocks go from global memory straight into LDS (buffer_load ... lds, no staging registers).  Two workgroups
// share a CU, so one workgroup's matrix work fills the other's waits (at head size 256 and B = 128 its 128 KiB of
// buffers leave room for one).
//
// Long calls are bound by power: with all inputs zero the same launches take 0.7 of their time, at a clock of 2.4 instead of
// 1.5 to 1.7 GHz.  What takes instructions, operand traffic or energy per operation out therefore shows in the run time,
// and what only fills idle cycles shows less.
//
// LDS layouts (rows of 2 D bytes, unpadded: the direct loads write 1 KiB contiguously): K has its
// 16-byte chunks XORed with (row & 15), so the 16 rows a quarter-wave reads one chunk of spread
// over all banks; V has its 32-byte groups XORed with row bits, which does the same for the rows of a transposing read.  At D = 64 two 128-byte rows share the 64 banks, so the row's bit 0 is left out of the
// terms.  The swizzle is applied on the global side (each lane fetches the chunk that belongs at its LDS position).
#include <type_traits>
#include <utility>

#include "stem_common.h"

namespace stem {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2_t;
typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2_t;
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4_t;
typedef __attribute__((address_space(3))) void lds_void_t;
typedef __attribute__((address_space(3))) s16x4_t lds_s16x4_t;

__device__ __forceinline__ u32x4_t as_u32x4(uint4 x) { return u32x4_t{x.x, x.y, x.z, x.w}; }
__device__ __forceinline__ bf16x8_t as_bf16x8(u32x4_t x) { return __builtin_bit_cast(bf16x8_t, x); }

__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
    f32x2_t f = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2_t));
}

// Larger of three, ignoring NaN.  (Written out: for fmaxf the compiler first quiets each matrix result with an
// instruction of its own, three vector instructions per pair of scores instead of one.)
__device__ __forceinline__ float max3(float a, float b, float c) {
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// Lanes whose query (16-query tile, lane % 16) lies before key 4 (lane / 16) + x of the 16 keys on the diagonal
constexpr uint64_t lanes_before_key(int x) {
    uint64_t lanes = 0;
    for (int l = 0; l < 64; ++l)
        if (4 * (l / 16) + x > l % 16) lanes |= 1ull << l;
    return lanes;
}

// f(0), f(1), .. f(N - 1) with compile-time arguments: what is inside is unrolled by the front end, whatever its size
template <typename F, int... I>
__device__ __forceinline__ void for_each_constant(std::integer_sequence<int, I...>, F&& f) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void unrolled(F&& f) {
    for_each_constant(std::make_integer_sequence<int, N>{}, f);
}
#define STEM_INLINE __attribute__((always_inline))

// Workgroup barrier without the memory fence of __syncthreads (which would wait for every
// outstanding global->LDS load); the waits are placed by hand.
#define STEM_BARRIER()                              \
    do {                                            \
        asm volatile("" ::: "memory");              \
        __builtin_amdgcn_s_barrier();               \
        asm volatile("" ::: "memory");              \
    } while (0)
// s_waitcnt with only vmcnt set (gfx9 encoding: vmcnt[3:0], expcnt[6:4]=7, lgkmcnt[11:8]=15); the
// builtin, unlike inline asm, is seen by the compiler's own wait-count bookkeeping.  vmcnt is split over bits [3:0] and
// [15:14].
#define STEM_WAIT_VMCNT(N) __builtin_amdgcn_s_waitcnt(0x0F70 | ((N) & 15) | (((N) >> 4) << 14))
// the same with only lgkmcnt set
#define STEM_WAIT_LGKMCNT_CASE(N) case N: __builtin_amdgcn_s_waitcnt(0xC07F | ((N) << 8)); break;
__device__ __forceinline__ void wait_lgkmcnt(int n) {   // n is a constant after unrolling: the switch folds away
    switch (n) {
        STEM_WAIT_LGKMCNT_CASE(0) STEM_WAIT_LGKMCNT_CASE(1) STEM_WAIT_LGKMCNT_CASE(2) STEM_WAIT_LGKMCNT_CASE(3)
        STEM_WAIT_LGKMCNT_CASE(4) STEM_WAIT_LGKMCNT_CASE(5) STEM_WAIT_LGKMCNT_CASE(6) STEM_WAIT_LGKMCNT_CASE(7)
        STEM_WAIT_LGKMCNT_CASE(8) STEM_WAIT_LGKMCNT_CASE(9) STEM_WAIT_LGKMCNT_CASE(10) STEM_WAIT_LGKMCNT_CASE(11)
        STEM_WAIT_LGKMCNT_CASE(12) STEM_WAIT_LGKMCNT_CASE(13) STEM_WAIT_LGKMCNT_CASE(14)
        default: break;
    }
}

// Nothing is scheduled across this point: keeps the next group of LDS operand reads ahead of the
// matrix instructions that consume the current group, operand reads in the order of their use, and a matrix
// instruction ahead of the softmax steps that go under it.
#define STEM_SCHED_FENCE() __builtin_amdgcn_sched_barrier(0)

// O^T += V^T P^T, 16 x 16 tile, 32 keys.  Written out because the compiler's form for four result registers lets the
// result land in other registers than the addend: over a branch that rescales O (the slow path of the softmax) it then
// copied all of O, on the common path too.  What the compiler does not know for such an instruction is kept by the code
// around it and checked in the finished assembly (wait_states.py): 8 issue slots before a vector access to the result.
template <bool ACC>
__device__ __forceinline__ void mfma_output(f32x4_t& c, u32x4_t a, u32x4_t b) {
    if constexpr (ACC) asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
    else asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
}
// Idle issue slots between the instructions that wrote o and vector instructions that touch it.  (Every register is named as
// one that the wait modifies: only that dependence keeps the compiler from moving the others across it.)
// (ACC: o lies in accumulator registers.)
template <int N, bool ACC, int M, int Q>
__device__ __forceinline__ void wait_states_output(f32x4_t (&o)[M][Q]) {
    auto here = [&]() STEM_INLINE {
#pragma unroll
        for (int x = 0; x < M * Q; ++x) {
            if constexpr (ACC) asm volatile("" : "+a"(o[x / Q][x % Q]));
            else asm volatile("" : "+v"(o[x / Q][x % Q]));
        }
    };
    here();
    asm volatile("s_nop %0" : : "n"(N - 1));
    here();
}

// Pins a Q operand to accumulator registers where it is loaded (kAcc, sparse_attn_body).
__device__ __forceinline__ void pin_to_acc(u32x4_t& x) { asm volatile("" : "+a"(x)); }

// One 1 KiB slice (1024 / 2D rows) of a B x D bf16 block, global -> LDS.  A block is D / 16 slices
// per wave: wave w issues slices u*NW + w, so that the row's swizzle term depends on u with a short
// period only (1, 2 or 4).  Requests are issued one at a time between matrix
// instructions, never as a burst: the texture-address unit takes a wave's 1 KiB request at
// 64 B/clk, and a wave that finds its queue full cannot issue anything else.
//
// The loads use buffer addressing with one resource per tensor and workgroup: its base is the
// sequence's first row in this KV head and its size ends with the sequence's last row, so rows
// past the end of a partial last block (and past the end of the tensor) are never read and arrive
// in LDS as zeros (their keys are masked by causality, their values get weight 0).  A block is a
// byte offset added to the per-lane offset (one vector add per block); the slice's offset, which
// is the same for all lanes, travels in the load's scalar offset operand, which the range check
// of a raw buffer takes into account (offset >= num_records - scalar offset reads as zero).
template <int NV>
struct BlockRequest {
    __amdgpu_buffer_rsrc_t rsrc;
    uint32_t lane_off[NV];          // block offset + per-lane byte offset, for u % NV (the swizzle term of a
                                    // slice's rows repeats with period NV = 1, 2 or 4 in u)

    __device__ __forceinline__ void issue(int u, unsigned char* __restrict__ slice0, uint32_t slice_step,
                                          int slice_lds_step) const {
        // slice0 = LDS address of this wave's slice for u = 0; slice u lies u*NW KiB further on
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void_t*)(slice0 + u * slice_lds_step), 16,
                                                 lane_off[u % NV], u * slice_step, 0, 0);
    }
};

// raw buffer (stride 0): num_records in bytes, loads beyond it return zero; 0x00020000 is the
// gfx9-family descriptor word for untyped 32-bit data
__device__ __forceinline__ __amdgpu_buffer_rsrc_t sequence_resource(const uint16_t* first_row, int rows,
                                                                    int64_t row_bytes, int head_bytes) {
    const int64_t bytes = rows > 0 ? (int64_t)(rows - 1) * row_bytes + head_bytes : 0;   // < 2^31 (host check)
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(first_row), 0, (int)bytes, 0x00020000);
}

// The order in which the query-block rows of a packed batch are handed out (launch_sparse_attn says when): the
// sequences by the length of their longest list's bound (the block index of the last row), longest first, and a
// sequence's rows from the last to the first, so that what starts last is short.  Packed as they come, a batch
// of short prompts can leave its longest row for the end.
struct RowWalk {
    int32_t start[STEM_MAX_BATCH];                     // prefix sums of the rows of the sequences in this order, then R
    uint8_t seq[STEM_MAX_BATCH];
};
// one sequence; several, rows from the last of the call to the first; several, in the walk's order
enum RowOrder : int { kOneSequence, kAsPacked, kWalk };

// Workgroup id -> XCD is id % 8 and cannot be changed once launched, and the XCDs of a chip are not equally fast
// under this kernel: given an eighth of the rows each, the last one ends 3 to 4.5 % after the mean (128K: 9.09 to 9.69 ms).
// So in long launches the last eighth or quarter of every XCD's rows is not handed out by workgroup id: the
// workgroups from slot `claim_from` on claim theirs when they start, from their own XCD's queue as long as it has
// rows, then from the one with most left.  There are a quarter more such workgroups than rows, so that a fast XCD can
// take more than its share; who finds nothing returns.  A claim is one atomic addition (taken[x * kQueueStride]: rows of
// XCD x claimed so far) with a look at the other counters in flight beside it.  Which workgroup takes a row has no
// influence on the row's result.
constexpr int kQueueStride = 32;                       // a 128-byte line each
static_assert(8 * kQueueStride * sizeof(int32_t) == STEM_ATTN_QUEUE_BYTES, "one line per XCD");

// The claim of one wave.  rows_of(x): how many rows XCD x has beyond claim_from (<= 0: none).  Sets xcd and slot;
// false if all queues are empty.  Every turn of the loop that does not end it finds one more queue used up, for good.
template <typename Rows>
__device__ __forceinline__ bool claim_row(int32_t* taken, int claim_from, Rows rows_of, int& xcd, int& slot) {
    const int lane = threadIdx.x & 63, x = lane & 7;
    const int rows = rows_of(x);
    for (int from = xcd;;) {
        int got = 0;
        if (lane == 0) got = __hip_atomic_fetch_add(taken + from * kQueueStride, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const int left = rows - __hip_atomic_load(taken + x * kQueueStride, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const int n = __builtin_amdgcn_readfirstlane(got);
        if (n < __builtin_amdgcn_readlane(rows, from)) {
            xcd = from;
            slot = claim_from + n;
            return true;
        }
        int most = 0, next = -1;
        for (int y = 0; y < 8; ++y) {
            const int l = __builtin_amdgcn_readlane(left, y);
            if (y != from && l > most) { most = l; next = y; }
        }
        if (next < 0) return false;
        from = next;
    }
}

// All queues at the start of a launch.  (A kernel and not a memset, which a captured graph would not replay reliably.)
__global__ void clear_row_queues_kernel(int32_t* taken) { taken[threadIdx.x * kQueueStride] = 0; }

// The row of a workgroup
struct RowPlace {
    int g, h;                                          // KV head, query head
    int r, i;                                          // row of the call, block index in its sequence
    int seq_lo, seq_hi;                                // key token rows the call may read
    int tok_q0, q_hi;                                  // its first query token (Q, O and lse hold the chunk's tokens only), end of the sequence's
};

// Which (head, row): consecutive workgroup ids go to different XCDs (each with its own L2), so an XCD should see few KV
// heads, and all XCDs equal work.  With xcds_per_kv_head = m > 0 (Hkv divides 8) XCD x serves KV head x / m and every
// m-th row of it, rows descending (long rows first), the G heads of a group side by side; otherwise every XCD takes a
// contiguous range of the (KV head, row descending, head in group) order.  false: no row.  claimed: two words of LDS that
// are not in use yet.
template <int B, bool WALK>
__device__ __forceinline__ bool find_row(const SeqTable& seq, const RowWalk& walk, int Hq, int R, int G, int order,
                                         int claim_from, int items_per_xcd, int xcds_per_kv_head,
                                         int32_t* __restrict__ taken, int* claimed, RowPlace& p) {
    int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    if (__builtin_expect(slot >= claim_from, 0)) {     // (travels beside `order`)
        if (threadIdx.x < 64) {
            const bool found = claim_row(taken, claim_from, [&](int x) {
                return rows_of_xcd(x, Hq, R, G, items_per_xcd, xcds_per_kv_head) - claim_from;
            }, xcd, slot);
            if (threadIdx.x == 0) {
                claimed[0] = found ? xcd : -1;
                claimed[1] = slot;
            }
        }
        __syncthreads();
        xcd = __builtin_amdgcn_readfirstlane(claimed[0]);
        slot = __builtin_amdgcn_readfirstlane(claimed[1]);
        __syncthreads();
        if (xcd < 0) return false;
    }
    int pos;                                           // place of the row in the walk
    if (xcds_per_kv_head > 0) {
        pos = (slot / G) * xcds_per_kv_head + xcd % xcds_per_kv_head;
        if (slot >= items_per_xcd || pos >= R) return false;
        p.g = xcd / xcds_per_kv_head;
        p.h = p.g * G + slot % G;
    } else {
        const int64_t item = (int64_t)xcd * items_per_xcd + slot;
        if (slot >= items_per_xcd || item >= (int64_t)Hq * R) return false;
        p.g = (int)(item / ((int64_t)R * G));
        const int rem = (int)(item - (int64_t)p.g * R * G);
        pos = rem / G;
        p.h = p.g * G + rem % G;
    }

    // The row comes first: its count and list entries are what everything else waits for.  `order` travels
    // beside R, so that a call of one sequence waits for no load here.  In the walk's order the sequence and its
    // place are found as in place_in, by a load per lane of either.
    int r = R - 1 - pos, s = 0;
    if (WALK && order == kWalk) {
        const int x = threadIdx.x & 63;
        const int start_x = walk.start[x], seq_x = walk.seq[x];
        const int turn = (int)__popcll(__builtin_amdgcn_ballot_w64(start_x <= pos)) - 1;
        s = __builtin_amdgcn_readlane(seq_x, turn);
        r = seq.row_start[s + 1] - 1 - (pos - __builtin_amdgcn_readlane(start_x, turn));
    } else if (order == kAsPacked) {
        s = seq_of_row(seq, r);
    }
    const int ic = r - seq.row_start[s];               // row inside the call's chunk of the sequence
    p.r = r;
    p.i = seq.first_block[s] + ic;
    p.seq_lo = seq.tok_start[s];
    p.seq_hi = seq.kv_end[s];
    p.tok_q0 = seq.q_tok_start[s] + ic * B;
    p.q_hi = seq.q_tok_start[s + 1];
    return true;
}

// Products of 16 x 16 x 32: at the power limit this instruction gives a ninth more operations per
// second than 32 x 32 x 16 (registers only 2020 / 1800 TFLOP/s, with the LDS reads and exponentials of this kernel beside it
// 1710 / 1540; with all inputs zero both reach 2440), and with two tiles of 16 queries per wave an LDS operand feeds as many
// operations.  Lane l has query l % 16 of each of the wave's QW tiles and, of 16 keys, the four from 4 (l / 16) on; two such
// key tiles are what the second product takes from a lane.  (QW: see launch_sparse_attn.)
//
// A block is worked on in halves of B / 2 keys, and the three steps of consecutive halves overlap.  Phase p is
//     S^T of half p, under it the second half of the softmax of half p - 1;
//     the reference check of half p - 1;
//     O^T of half p - 1, under it the first half of the softmax of half p,
// so that every matrix instruction has the same share of the softmax beside it (all of a block's under its last tile and a half of
// S^T and first of O^T before: two waves of a SIMD in that part at once left the matrix pipe idle).  The LDS operands of the
// two products are one stream that is read kAhead operands ahead, across phases too; K and V have two buffers each, one per half,
// and where the stream goes on to the next phase the wave waits for the requests that fill it and for the others to have
// read what the next phase's requests overwrite: one barrier per half block.  These requests are issued during S^T (kTail: before
// it).  A row's first half has its whole softmax at its check, from references that look into the second (kPastHalf).
//
// Before (32 x 32 x 16, softmax under the same block's products) / now, attention alone: 128K, 8 % of the blocks 9234 / 8494 us;
// 64K, all 24393 / 22345; 32K, 15 % 1114 / 1035; 64K, 5 % 1315 / 1245; d = 64, 64K 1405 / 1332; 12 prompts to 2047 tokens 119 / 114, d = 64
// 73.3 / 71.6; B = 64, 4096 tokens of one head 14.0 / 12.7, 100K tokens 7622 / 7603 and d = 64, 50K 1079 / 1056.
//
// Head size 256.  A wave of 32 queries needs 440 (B = 64: 408) registers, so it has its SIMD for itself, and half of them are
// accumulator registers, which only matrix instructions and copies can reach (kAcc): O and Q lie there, everything that the
// softmax touches in vector registers.  Left to itself the compiler placed the scores there as well, or O in vector registers and
// copied other values back and forth, 116 copies per block (32K, 15 %: 2587 us; by a flag for this file the results of the
// other matrix instructions stay in vector registers, which alone gave 2491).  With 16 queries a wave needs 200, and two share a SIMD;
// each LDS operand then feeds one matrix instruction.  Before (32 x 32 x 16, one wave per SIMD, the softmax under the same
// block's products, two barriers per block) / now, attention alone, B = 128: 32K, 15 % 2298 / 2104 us; 115 blocks, 54 of them kept
// 2094 / 1889; 12 prompts to 2047 tokens 260 / 233; B = 64: 203 blocks, 54 kept 1208 / 1120.
//
// LDS there: 128 KiB at B = 128, where the immediate offset of a read reaches 64 KiB.  With K below and V from 64 KiB on the second
// half of V took two more vector instructions for every read, 62 per block, with nobody on the SIMD to fill them in.  So V lies
// below, and the distance to K is in a lane's base, which the bases of a half's reads are formed from anyway.  Attention alone
// before / now: 228 rows of 100 blocks 302 / 273 us (32 x 32 x 16 products 294), 64 of 50 137 / 131 (134), 3072 of 20 768 / 740.
//
// Every query's arithmetic is its 16-query tile's own: a reference moves for a tile at a time, and no step depends on
// how many tiles share a wave.
template <int B, int D>
constexpr bool kKeysBeyondOffset = 4 * B * D > 65536;
template <int B, int D, int QW>
__device__ __forceinline__ void sparse_attn_body(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    const int32_t* __restrict__ counts, const int32_t* __restrict__ indices, uint16_t* __restrict__ out,
    float* __restrict__ lse, const RowPlace& row, int R, int T, int kmax, bool shared_lists, int64_t q_st, int64_t q_sh,
    int64_t kv_st, int64_t kv_sh, float scale, unsigned char* __restrict__ k_lds_a, unsigned char* __restrict__ k_lds_b,
    unsigned char* __restrict__ v_lds_a, unsigned char* __restrict__ v_lds_b) {
    // (where K lies beyond the immediate offset its parameters are kKeysAt short of it)
    // (a parameter of its own for every buffer: alias-scope information then tells the compiler's wait-count insertion a
    // read of one buffer from a request in flight into another; otherwise it waits for all of them)
    constexpr int KT = B / 32;                         // 32-key tiles per block
    constexpr int KS = D / 16;                         // LDS operands of a tile, in either product
    constexpr int KD = D / 32;                         // 32-wide steps of S^T along d
    constexpr int NW = B / (16 * QW);                  // waves
    constexpr int KR = D * QW / 32;                    // requests per wave, tensor and block
    constexpr int TP = KT / 2;                         // tiles per half block
    constexpr int HS = TP * KS;                        // LDS operands of a half block, in either product
    constexpr int NP = TP * 4 * QW;                    // softmax pairs per lane and half block
    constexpr int kKeysAt = kKeysBeyondOffset<B, D> ? 2 * B * D : 0;   // (sparse_attn_kernel)
    constexpr bool kAcc = D == 256 && QW == 2;         // O and Q in accumulator registers
    constexpr int kRowBytes = D * 2;                   // one K or V row in LDS
    constexpr int kSliceRows = 1024 / kRowBytes;       // rows one wave-wide 1 KiB request covers
    // LDS swizzles, as XORs on the 16-byte chunk index of a row: K spreads the 16 rows a quarter-wave reads one chunk of over
    // all banks, V the 8 rows x 32 bytes of half a transposing read (at d = 64 two 128-byte rows share the 64 banks)
    auto k_swz = [](int row) { return D == 64 ? (row >> 1) & 7 : row & 15; };
    auto v_swz = [](int row) { return (D == 64 ? (row >> 1) & 3 : row & 7) << 1; };
    using C0 = std::integral_constant<int, 0>;
    using C1 = std::integral_constant<int, 1>;

    const int i = row.i;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int w_tile = w * QW / 2;                     // the 32-key tile that holds the keys on this wave's diagonal
    const int c16 = lane & 15, grp = lane >> 4;

    const int64_t list_row = (int64_t)(shared_lists ? row.g : row.h) * R + row.r;   // whose list: the KV head's or the query head's
    const int32_t* list = indices + list_row * kmax;
    // the first 64 entries without waiting for the count (a row has room for kmax; what lies beyond the count is
    // clamped where it is used as an address, and never used otherwise)
    int list_reg = lane < kmax ? list[lane] : 0;
    const int cnt = min(counts[list_row], kmax);

    // ---- Q rows of this wave as B operands: per tile, KD steps of 32 along d.  Queries past the end repeat the last one (no
    //      branch around a load); what they give is not stored ----
    u32x4_t q_reg[QW][KD];
#pragma unroll
    for (int qt = 0; qt < QW; ++qt) {
        const uint16_t* src = q + (int64_t)min(row.tok_q0 + (w * QW + qt) * 16 + c16, row.q_hi - 1) * q_st +
                              (int64_t)row.h * q_sh + grp * 8;
#pragma unroll
        for (int ks = 0; ks < KD; ++ks) q_reg[qt][ks] = as_u32x4(*reinterpret_cast<const uint4*>(src + ks * 32));
    }

    // per-lane byte offsets of the block requests (BlockRequest): slice u of wave w is the 1 KiB at LDS offset
    // (u NW + w) KiB of the block; lane l writes chunk pc of row (u NW + w) kSliceRows + slice_row there and fetches the chunk
    // that belongs at that position, i.e. the swizzle is applied to the global column.  Only the low bits of the row
    // enter the swizzle, so it repeats in u with a short period.
    const int64_t row_bytes = kv_st * 2;
    const int slice_row = (lane * 16) / kRowBytes, pc = ((lane * 16) % kRowBytes) >> 4;
    const int lrow = w * kSliceRows + slice_row;       // row of slice u = 0
    const uint32_t lane_row_off = (uint32_t)(lrow * row_bytes);
    constexpr int kKVariants = D >= 128 && NW * kSliceRows < 16 ? 16 / (NW * kSliceRows) : 1;
    static_assert((kKVariants * NW * kSliceRows) % 16 == 0, "the K swizzle term of slice u repeats with period kKVariants");
    constexpr int kVVariants = NW * kSliceRows < 8 ? 8 / (NW * kSliceRows) : 1;
    static_assert((kVVariants * NW * kSliceRows) % 8 == 0, "the V swizzle term of slice u repeats with period kVVariants");
    uint32_t k_off[kKVariants];
#pragma unroll
    for (int x = 0; x < kKVariants; ++x) k_off[x] = lane_row_off + ((pc ^ k_swz(lrow + x * NW * kSliceRows)) << 4);
    uint32_t v_off[kVVariants];
#pragma unroll
    for (int x = 0; x < kVVariants; ++x) v_off[x] = lane_row_off + ((pc ^ v_swz(lrow + x * NW * kSliceRows)) << 4);
    const int64_t first_row = (int64_t)row.g * kv_sh + (int64_t)row.seq_lo * kv_st;
    const auto k_rsrc = sequence_resource(k + first_row, row.seq_hi - row.seq_lo, row_bytes, kRowBytes);
    const auto v_rsrc = sequence_resource(v + first_row, row.seq_hi - row.seq_lo, row_bytes, kRowBytes);
    const uint32_t block_bytes = (uint32_t)(B * row_bytes);
    const uint32_t slice_step = (uint32_t)(NW * kSliceRows * row_bytes);   // rows of slices u and u+1 of one wave
    constexpr int slice_lds_step = NW * 1024;
    auto k_request = [&](int j, bool wanted = true) {  // not wanted: beyond the resource, nothing is fetched
        const uint32_t off = wanted ? j * block_bytes : 0x80000000u;
        BlockRequest<kKVariants> rq{k_rsrc, {}};
#pragma unroll
        for (int x = 0; x < kKVariants; ++x) rq.lane_off[x] = k_off[x] + off;
        return rq;
    };
    auto v_request = [&](int j) {
        BlockRequest<kVVariants> rq{v_rsrc, {}};
#pragma unroll
        for (int x = 0; x < kVVariants; ++x) rq.lane_off[x] = v_off[x] + j * block_bytes;
        return rq;
    };
    // the first KR / 2 requests of a block are its first half
    auto issue_k = [&](const BlockRequest<kKVariants>& rq, int u) {
        rq.issue(u, (u < KR / 2 ? k_lds_a : k_lds_b - (KR / 2) * slice_lds_step) + kKeysAt + w * 1024, slice_step, slice_lds_step);
    };
    auto issue_v = [&](const BlockRequest<kVVariants>& rq, int u) {
        rq.issue(u, (u < KR / 2 ? v_lds_a : v_lds_b - (KR / 2) * slice_lds_step) + w * 1024, slice_step, slice_lds_step);
    };

    // List entries outside 0..i break the precondition; they are processed as fully masked
    // blocks (clamped for addressing), which costs time but keeps the control flow flat.
    auto usable = [&](int j) { return j >= 0 && j <= i; };
    auto clamped = [&](int j) { return min(max(j, 0), i); };
    // The list lives in a vector register, 64 entries at a time (lane e holds entry e of the
    // chunk), and entries are taken out with v_readlane: no scalar load sits in the loop, so the
    // in-order LDS operand reads are the only users of their counter there.
    auto list_chunk = [&](int first) {                 // (lane from its number: no register holds an address through the blocks)
        const int e = first + __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
        return e < cnt ? list[e] : 0;
    };
    int j_cur = __builtin_amdgcn_readlane(list_reg, 0);
    {                                                  // (an empty list: a block that nothing uses)
        const auto rk = k_request(clamped(j_cur));
        const auto rv = v_request(clamped(j_cur));
#pragma unroll
        for (int u = 0; u < KR; ++u) issue_k(rk, u);
#pragma unroll
        for (int u = 0; u < KR / 2; ++u) issue_v(rv, u);
    }

    // The output pointers are taken now: a scalar load still in flight would make every wait for LDS operands in the
    // blocks one for all of them (the two kinds return in any order on one counter).
    asm volatile("" : : "s"(out), "s"(lse));

    if constexpr (kAcc) {
#pragma unroll
        for (int x = 0; x < QW * KD; ++x) pin_to_acc(q_reg[x / KD][x % KD]);
    }
    const f32x4_t zero4 = {0.f, 0.f, 0.f, 0.f};
    f32x4_t o_acc[KS][QW];                             // [16-column tile][query tile]
#pragma unroll
    for (int x = 0; x < KS * QW; ++x) o_acc[x / QW][x % QW] = zero4;
    const float neg_inf = -__builtin_huge_valf();
    const float sl2 = scale * 1.4426950408889634f;
    f32x4_t l_win[QW];                                 // row sums of the current half (four equal copies)
    float m_ref[QW], off[QW], l_run[QW];               // softmax reference (raw score units) and, negated, in exp2 units; sum
#pragma unroll
    for (int qt = 0; qt < QW; ++qt) {
        m_ref[qt] = neg_inf;
        off[qt] = l_run[qt] = 0.f;
        l_win[qt] = zero4;
    }
    // The first references are the largest scores of the first 96 keys of a row, at B = 64 of the first 32: what they are taken from
    // decides how every probability rounds, and the largest, being 1, does not.  (From the first 64 at B = 128 lse was up to 1.3 times
    // as far from 64 bits, and the outputs 1 %.  The softmax of a row's first half has nothing to go under this way: attention alone,
    // 64 / 96 keys, 12 prompts to 2047 tokens 96.8 / 97.2 us, d = 64 62.1 / 62.8; 128 rows of 8 blocks 16.7 / 16.9; 128K the same.)
    constexpr bool kPastHalf = B == 128;
    bool first = kPastHalf;                          // no query has a reference yet: the first half is left to fix_half
    bool unseen = kPastHalf;                         // a query has no reference yet: all it has met is masked

    // per-lane LDS offsets that do not change between blocks.  Both swizzles are XORs of address
    // bits that are zero in the unswizzled per-lane offset, so the offset of an operand is one
    // v_xor of a per-lane base with a constant, plus an immediate.
    uint32_t k_base = c16 * kRowBytes + ((k_swz(c16) ^ grp) << 4);
    if constexpr (kKeysAt > 0) {
        k_base += kKeysAt;
        asm("" : "+v"(k_base));                        // stays in the base: the rest is a constant within the immediate offset
    }
    // transposing V read: lane l fetches row 4 (l / 16) + (l % 16) / 4 of 16 rows, 8 bytes at column 16 dt + 4 (l % 4)
    const int v_row = grp * 4 + (c16 >> 2);
    const uint32_t v_base = v_row * kRowBytes + (v_swz(v_row) << 4) + ((lane & 3) << 3);
    // Operand n of S^T of half P: tile n / KS, 16 keys n % 2 of it, 32-wide step (n % KS) / 2 along d; and of O^T: tile n / KS,
    // 16 columns n % KS (the tile's 32 keys in two reads).
    auto load_k = [&](int P, int n) {
        const int t = n / KS, kt = n & 1, ks = (n % KS) >> 1;
        return *reinterpret_cast<const u32x4_t*>((P ? k_lds_b : k_lds_a) + (k_base ^ (ks << 6)) + (t * 32 + kt * 16) * kRowBytes);
    };
    auto load_v = [&](int P, int n) {
        const int t = n / KS, dt = n % KS;
        const unsigned char* p0 = (P ? v_lds_b : v_lds_a) + (v_base ^ (dt << 5)) + t * 32 * kRowBytes;
        const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)p0);
        const s16x4_t up = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)(p0 + 16 * kRowBytes));
        const uint2 lo2 = __builtin_bit_cast(uint2, lo), up2 = __builtin_bit_cast(uint2, up);
        return u32x4_t{lo2.x, lo2.y, up2.x, up2.y};
    };
    // Operands are read this many ahead of their use, and used two at a time behind one wait.  Attention alone, 4 / 2 ahead:
    // 128K 8716 / 8698 us, 5 % 1285 / 1279, 32K 1066 / 1064, B = 64 100K 7725 / 7687 (and six 3 to 4 % slower than four).  With one
    // tile per wave an operand is used up in half the time: 4 / 6 / 8 ahead one head of 4096 (B = 64) 12.3 / 11.7 / 11.8, 25 rows of
    // 12 blocks (B = 128) 35.8 / 35.7 / 34.9, and, with kTail, 6 / 8 ahead at B = 64 64 rows of 60 blocks far away 64.3 / 62.6; at d = 256, 2 / 4 / 6 / 8 ahead, 32K 2435 / 2451 / 2456 / 2457.  B = 128, d = 64 has a
    // half block's products done in eight operands: read eight ahead the wait for the next phase's requests came right behind
    // these.  2 / 4 / 6 / 8, 64 rows of 50 blocks 55.8 / 56.3 / 56.5 / 58.6 us, 228 of 100 109 / 110 / 112 / 117 (32 x 32 x 16 products 56.2, 112).
    constexpr int kWanted = QW == 1 && D != 256 ? (B == 128 && D == 64 ? 2 : 8) : 2;
    constexpr int kAhead = kWanted < HS ? kWanted : HS;
    // The operand of S^T under which request u of a phase is issued, K's first.  B = 64 and d = 64, over all of S^T / its first
    // half: 100K 8185 / 7931 us, d = 64 1436 / 1431; 128K the other way round, 8994 / 9041.
    // d = 256, B = 64: two tiles per wave, 256 blocks of which 50 kept 1403 / 1365; one tile, 100 rows of 8 blocks 13.4 / 14.1.
    constexpr bool kEarly = (B == 64 || D == 64) && !(D == 256 && QW == 1);
    auto request_slot = [](int u) { return kEarly ? u * HS / (2 * KR) : u * HS / KR; };
    // kTail: a phase's requests go out in the phase before instead, one under each operand of O^T from where its reading side has
    // crossed into the next phase: from there on nobody reads the buffers that they fill, and they have a whole phase to arrive.
    // A row by itself at B = 64 waits for them otherwise where its keys are not in the L2.  64 rows, in late chunks of 64K tokens / of
    // few keys, 32 x 32 x 16 products / before / now: d = 64, 60 blocks 51.4 / 59.1 / 53.6 us and 36.5 / 33.7 / 33.6 (50 blocks); d = 128 60.1 /
    // 66.4 / 62.6 and 47.3 / 41.4 / 40.6.  Two at a time or all at once 1 to 6 % slower.
    constexpr bool kTail = QW == 1 && B == 64 && D != 256;
    static_assert(!kTail || KR <= kAhead, "an operand for every request");

    f32x4_t s_acc[2][TP][2][QW];                       // [half][tile][16 keys][query tile]
    u32x4_t p_pk[2][TP][QW];                           // bf16 pairs: [half][tile][query tile], [2 * 16 keys + pair]
    float f0 = 0.f, f1 = 0.f;                          // the pair in flight
    const uint32_t one2 = 0x3f803f80u;
    u32x4_t ones = {one2, one2, one2, one2};
    // (kept in vector registers instead of moved there for every use: 128K 8698 / 8684 us, d = 64 1383 / 1377; B = 64 100K 7687 / 7740)
    if constexpr (B == 128) asm volatile("" : "+v"(ones));

    // Step u % 4 of softmax pair u / 4 of half P: exponents, two exponentials, packing to bf16.  The row sums are taken from the
    // rounded values by the matrix pipe, a tile's 32 keys at a time: a product of the tile's P^T operand with ones, which
    // gives every lane the sum of its own query.  It is issued a step into the next pair (at the end of a run of pairs at once),
    // so that it does not wait for the packing (128K 8684 / 8659 us).
    auto row_sum = [&](auto P_tag, auto pair_tag) STEM_INLINE {     // of the four pairs that end with this one
        constexpr int P = decltype(P_tag)::value, pair = decltype(pair_tag)::value, t = pair / (4 * QW), qt = (pair >> 2) % QW;
        l_win[qt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(ones), as_bf16x8(p_pk[P][t][qt]), t == 0 ? zero4 : l_win[qt],
                                                           0, 0, 0);
    };
    auto softmax_step = [&](auto P_tag, auto u_tag) STEM_INLINE {
        constexpr int P = decltype(P_tag)::value, u = decltype(u_tag)::value, pair = u >> 2;
        constexpr int t = pair / (4 * QW), qt = (pair >> 2) % QW, kt = (pair >> 1) & 1, x = (pair & 1) * 2;
        // (an opaque use of each result: without it the compiler gathers the softmax next to the consumer of the
        // probabilities instead of leaving each step under its matrix instruction)
        if constexpr ((u & 3) == 0) {
            f0 = __builtin_fmaf(s_acc[P][t][kt][qt][x], sl2, off[qt]);
            f1 = __builtin_fmaf(s_acc[P][t][kt][qt][x + 1], sl2, off[qt]);
            asm volatile("" : "+v"(f0), "+v"(f1));
        } else if constexpr ((u & 3) == 1) {
            if constexpr ((pair & 3) == 0 && pair > 0 && pair != NP / 2) row_sum(P_tag, std::integral_constant<int, pair - 1>{});
            f0 = __builtin_amdgcn_exp2f(f0);
            asm volatile("" : "+v"(f0));
        } else if constexpr ((u & 3) == 2) {
            f1 = __builtin_amdgcn_exp2f(f1);
            asm volatile("" : "+v"(f1));
        } else {
            uint32_t pk = pack_bf16(f0, f1);
            asm volatile("" : "+v"(pk));
            p_pk[P][t][qt][pair & 3] = pk;
            if constexpr ((pair & 3) == 3 && (pair == NP - 1 || pair == NP / 2 - 1)) row_sum(P_tag, std::integral_constant<int, pair>{});
        }
    };
    // pairs first .. first + N - 1, one after the other
    auto softmax_pairs = [&](auto P_tag, auto first, auto N) STEM_INLINE {
        unrolled<4 * decltype(N)::value>([&](auto u) STEM_INLINE {
            softmax_step(P_tag, std::integral_constant<int, 4 * decltype(first)::value + decltype(u)::value>{});
        });
    };
    // the steps of these pairs that go under matrix instruction `at` of the `span` that share them: step u to
    // (u + 1) span / n, so that no step waits for the one before it, the last one to the last
    auto softmax_under = [&](auto P_tag, auto first, auto N, auto at_tag, auto span_tag) STEM_INLINE {
        constexpr int n = 4 * decltype(N)::value, span = decltype(span_tag)::value, at = decltype(at_tag)::value;
        constexpr int from = (at * n + span - 1) / span - 1, next = at == span - 1 ? n : ((at + 1) * n + span - 1) / span - 1;
        constexpr int lo = from < 0 ? 0 : from, hi = next < n ? next : n;
        if constexpr (at < span && lo < hi)
            unrolled<hi - lo>([&](auto u) STEM_INLINE {
                softmax_step(P_tag, std::integral_constant<int, 4 * decltype(first)::value + lo + decltype(u)::value>{});
            });
    };
    using kAll = std::integral_constant<int, NP>;
    using kHalf = std::integral_constant<int, NP / 2>;

    auto negated_offset = [&](int qt) { return m_ref[qt] == neg_inf ? 0.f : -m_ref[qt] * sl2; };   // 0: masked scores stay at exp2(-inf) = 0
    // largest score of the query in half P, of its first `tiles` tiles (all of its lanes get it), ignoring NaN
    auto half_max = [&](int P, int qt, int tiles) {
        float mx2[2] = {neg_inf, neg_inf};
#pragma unroll
        for (int t = 0; t < tiles; ++t)
#pragma unroll
            for (int kt = 0; kt < 2; ++kt) {
                mx2[0] = max3(mx2[0], s_acc[P][t][kt][qt][0], s_acc[P][t][kt][qt][1]);
                mx2[1] = max3(mx2[1], s_acc[P][t][kt][qt][2], s_acc[P][t][kt][qt][3]);
            }
        const float mx = max3(mx2[0], mx2[1], mx2[1]);
        const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
        const float y = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
        const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(y), __float_as_uint(y), false, false);
        return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
    };
    auto note_unseen = [&]() {
        bool none = m_ref[0] == neg_inf;
        if constexpr (QW == 2) none |= m_ref[1] == neg_inf;
        unseen = __builtin_amdgcn_ballot_w64(none) != 0;
    };
    // The slow path of a half: for a query tile that needs it, moves the references of the tile's queries up to their true
    // maximum where that is higher (rescaling O and l) and forms the half's probabilities anew.  Where sums are not finite
    // only if a query gains by it: one that has no reference, or probabilities far beyond its own (a sum over 2^16 of 128 keys
    // at most holds one over 2^9), and a finite score to go to.  A query that is NaN or inf for good comes here with
    // every half and leaves the others as they are.
    // The first half of a row comes here too (kPastHalf), its scores and, if `both`, the second half's being there.
    auto fix_half = [&](auto P_tag, bool both) STEM_INLINE {
        constexpr int P = decltype(P_tag)::value;
        if (kPastHalf && first) {                    // (a copy of the softmax: where paths meet here O is copied at d = 256)
            first = false;
#pragma unroll
            for (int qt = 0; qt < QW; ++qt) {
                const float mx = half_max(P, qt, TP);
                m_ref[qt] = both ? fmaxf(mx, half_max(1 - P, qt, 1)) : mx;
                off[qt] = negated_offset(qt);
                asm volatile("" : "+v"(off[qt]));      // not folded into the exponents: the bits of the common path
            }
            softmax_pairs(P_tag, C0{}, kAll{});
            note_unseen();
            return;
        }
        wait_states_output<16, kAcc>(o_acc);           // the last O^T instruction has written
        if constexpr (kAcc) asm volatile("" : "+v"(l_win[0]), "+v"(l_win[QW - 1]));   // and the last row sum's
#pragma unroll
        for (int qt = 0; qt < QW; ++qt) {
            const bool needs = __builtin_amdgcn_ballot_w64((m_ref[qt] == neg_inf) | !(l_win[qt][0] <= 65536.0f)) != 0;
            const float mx = half_max(P, qt, TP);
            const bool gains = (mx < -neg_inf) & (mx > m_ref[qt]) & ((m_ref[qt] == neg_inf) | (mx * sl2 + off[qt] > 8.9f));
            const bool moves = (__builtin_amdgcn_ballot_w64(!(l_win[qt][0] < -neg_inf)) == 0) | (__builtin_amdgcn_ballot_w64(gains) != 0);
            const bool up = needs & moves & (mx > m_ref[qt]);
            const float corr = !up ? 1.f : m_ref[qt] == neg_inf ? 0.f : __builtin_amdgcn_exp2f((m_ref[qt] - mx) * sl2);
            m_ref[qt] = up ? mx : m_ref[qt];
            l_run[qt] *= corr;
#pragma unroll
            for (int dt = 0; dt < KS; ++dt)
#pragma unroll
                for (int x = 0; x < 4; ++x) o_acc[dt][qt][x] *= corr;
            off[qt] = negated_offset(qt);
            asm volatile("" : "+v"(off[qt]));          // not folded into the exponents: the bits of the common path
        }
        softmax_pairs(P_tag, C0{}, kAll{});            // (those of a tile that stays come out as they were)
        wait_states_output<4, kAcc>(o_acc);            // before the next one reads them
        note_unseen();
    };
    // A half needs the slow path if a query has no reference yet or if its sum is not a modest finite number (a
    // probability above 2^16, inf, NaN: the reference is too low for this half).
    auto check_half = [&](auto P_tag, bool both = true) STEM_INLINE {
        // (the last sum's product has been issued just before; across the branches of the masks, which may lie in between, the
        // compiler kept four of the eight idle slots that its result needs at QW = 1, B = 128, and seven at QW = 2)
        if constexpr (QW == 1) asm volatile("s_nop 3" : "+v"(l_win[0]));
        else asm volatile("s_nop 0" : "+v"(l_win[1]));
        bool high = !(l_win[0][0] <= 65536.0f);
        if constexpr (QW == 2) high |= !(l_win[1][0] <= 65536.0f);
        if (unseen || __builtin_amdgcn_ballot_w64(high) != 0) fix_half(P_tag, both);
#pragma unroll
        for (int qt = 0; qt < QW; ++qt) l_run[qt] += l_win[qt][0];
    };
    // Masks the tiles of half P from `from` on: keys above the query on the diagonal block (w_tile and later), all keys of an
    // entry that cannot be used
    auto mask_half = [&](int P, int from, bool all) {
        const f32x4_t none = {neg_inf, neg_inf, neg_inf, neg_inf};
#pragma unroll
        for (int tt = 0; tt < TP; ++tt) {
            const int t = P * TP + tt;
            if (t < from) continue;
            auto diagonal = [&](f32x4_t& s) {          // 16 queries against the same 16 keys
#pragma unroll
                for (int x = 0; x < 4; ++x) s[x] = __builtin_amdgcn_inverse_ballot_w64(lanes_before_key(x)) ? neg_inf : s[x];
            };
            if (all || t > w_tile) {
#pragma unroll
                for (int x = 0; x < 2 * QW; ++x) s_acc[P][tt][x / QW][x % QW] = none;
            } else if constexpr (QW == 2) {
                s_acc[P][tt][1][0] = none;
                diagonal(s_acc[P][tt][0][0]);
                diagonal(s_acc[P][tt][1][1]);
            } else if (w & 1) {
                diagonal(s_acc[P][tt][1][0]);
            } else {
                s_acc[P][tt][1][0] = none;
                diagonal(s_acc[P][tt][0][0]);
            }
        }
    };
    auto block_mask = [&](int j, int& from, bool& all) {
        all = !usable(j);
        from = all ? 0 : j == i ? w_tile : KT;
    };

    // The matrix instructions of LDS operand m, `even` and `odd` being it and its partner of the pair m & ~1, m | 1.  With two query
    // tiles a pair's four instructions change one operand at a time.  under(h): what goes under the operand's h-th.
    auto scores = [&](auto P_tag, auto m_tag, u32x4_t even, u32x4_t odd, auto under) STEM_INLINE {
        constexpr int P = decltype(P_tag)::value, m = decltype(m_tag)::value, h = m & 1, t = m / KS, ks = (m % KS) >> 1;
        auto product = [&](f32x4_t& c, u32x4_t a, u32x4_t b) STEM_INLINE {
            c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(a), as_bf16x8(b), ks == 0 ? zero4 : c, 0, 0, 0);
            STEM_SCHED_FENCE();
        };
        if constexpr (QW == 2) {
            product(s_acc[P][t][h][h], h ? odd : even, q_reg[h][ks]);
            under(C0{});
            STEM_SCHED_FENCE();
            product(s_acc[P][t][1 - h][h], h ? even : odd, q_reg[h][ks]);
            under(C1{});
        } else {
            product(s_acc[P][t][h][0], h ? odd : even, q_reg[0][ks]);
            under(C0{});
        }
        STEM_SCHED_FENCE();
    };
    auto outputs = [&](auto P_tag, auto m_tag, u32x4_t even, u32x4_t odd, auto under) STEM_INLINE {
        constexpr int P = decltype(P_tag)::value, m = decltype(m_tag)::value, h = m & 1, t = m / KS, dt = (m % KS) & ~1;
        auto product = [&](f32x4_t& c, u32x4_t a, u32x4_t b) STEM_INLINE {
            mfma_output<kAcc>(c, a, b);
            STEM_SCHED_FENCE();
        };
        if constexpr (QW == 2) {
            product(o_acc[dt + h][h], h ? odd : even, p_pk[P][t][h]);
            under(C0{});
            STEM_SCHED_FENCE();
            product(o_acc[dt + 1 - h][h], h ? even : odd, p_pk[P][t][h]);
            under(C1{});
        } else {
            product(o_acc[dt + h][0], h ? odd : even, p_pk[P][t][0]);
            under(C0{});
        }
        STEM_SCHED_FENCE();
    };
    auto nothing = [](auto) {};
    // Where the reading side goes on to the next phase.  A wave's own reads have to be back before the others may ask for what
    // overwrites the buffer they read from.
    auto cross = [&]() {
        wait_lgkmcnt(0);
        STEM_WAIT_VMCNT(0);
        STEM_BARRIER();
    };
    auto waited = [&](int reads_behind) {
        wait_lgkmcnt(reads_behind);
        STEM_SCHED_FENCE();
    };
    u32x4_t ring[kAhead];                              // the first operands of the next phase
    using kSpan = std::integral_constant<int, QW * HS>;    // matrix instructions of either product in a phase

    // One phase: half P of a block, and O^T of the half before it.  request(m): the requests under operand m.
    auto phase = [&](auto P_tag, int mask_from, bool mask_all, auto request) STEM_INLINE {
        constexpr int P = decltype(P_tag)::value, Q = 1 - P;
        using Before = std::integral_constant<int, Q>;
        u32x4_t op[2 * HS + kAhead];
        unrolled<kAhead>([&](auto m) STEM_INLINE { op[m] = ring[m]; });
        unrolled<2 * HS>([&](auto m_tag) STEM_INLINE {
            constexpr int m = decltype(m_tag)::value;
            if constexpr ((m & 1) == 0) {
                constexpr int a = m + kAhead;
                if constexpr (a == 2 * HS) cross();
                op[a] = a < HS ? load_k(P, a) : a < 2 * HS ? load_v(Q, a - HS) : load_k(Q, a - 2 * HS);
                op[a + 1] = a < HS ? load_k(P, a + 1) : a < 2 * HS ? load_v(Q, a + 1 - HS) : load_k(Q, a + 1 - 2 * HS);
                // operands m + 2 .. a + 1 may be under way, those of O^T in two reads
                constexpr int v_lo = m + 2 > HS ? m + 2 : HS, v_hi = a + 2 < 2 * HS ? a + 2 : 2 * HS;
                if constexpr (a != 2 * HS) waited(kAhead + (v_hi > v_lo ? v_hi - v_lo : 0));
            }
            if constexpr (m < HS) {
                request(m);
                scores(P_tag, m_tag, op[m & ~1], op[m | 1], [&](auto h) STEM_INLINE {
                    softmax_under(Before{}, kHalf{}, kHalf{}, std::integral_constant<int, QW * m + decltype(h)::value>{}, kSpan{});
                });
                if constexpr (m == HS - 1) {
                    if (mask_from < KT) mask_half(P, mask_from, mask_all);
                    check_half(Before{});
                    STEM_SCHED_FENCE();
                }
            } else {
                request(m);
                outputs(Before{}, std::integral_constant<int, m - HS>{}, op[m & ~1], op[m | 1], [&](auto h) STEM_INLINE {
                    softmax_under(P_tag, C0{}, kHalf{}, std::integral_constant<int, QW * (m - HS) + decltype(h)::value>{}, kSpan{});
                });
            }
        });
        unrolled<kAhead>([&](auto m) STEM_INLINE { ring[m] = op[2 * HS + m]; });
    };

    if (cnt > 0) {
        int mask_from;
        bool mask_all;
        block_mask(j_cur, mask_from, mask_all);
        int j_nxt = kTail ? __builtin_amdgcn_readlane(list_reg, 1) : 0;
        STEM_WAIT_VMCNT(KR);                           // the first half of K is there (its second and V's first may not be)
        STEM_BARRIER();
        // ---- the first half: S^T alone; the references are its largest scores; the first half of its softmax ----
        {
            u32x4_t op[HS + kAhead];
            BlockRequest<kKVariants> rk;
            const auto rv = v_request(clamped(j_cur));
            unrolled<kAhead>([&](auto m) STEM_INLINE {
                op[m] = load_k(0, m);
                if (m & 1) STEM_SCHED_FENCE();
            });
            unrolled<HS>([&](auto m_tag) STEM_INLINE {
                constexpr int m = decltype(m_tag)::value, a = m + kAhead;
                if constexpr ((m & 1) == 0) {
                    if constexpr (a == HS) cross();
                    op[a] = a < HS ? load_k(0, a) : load_k(1, a - HS);
                    op[a + 1] = a < HS ? load_k(0, a + 1) : load_k(1, a + 1 - HS);
                    waited(kAhead);
                }
                if constexpr (kTail) {
                    if constexpr (m == HS - kAhead) rk = k_request(clamped(j_nxt), cnt > 1);
#pragma unroll
                    for (int u = 0; u < KR / 2; ++u) {
                        if (m == HS - kAhead + u) issue_k(rk, u);
                        if (m == HS - kAhead + u + KR / 2) issue_v(rv, u + KR / 2);
                    }
                }
                scores(C0{}, m_tag, op[m & ~1], op[m | 1], nothing);
            });
            unrolled<kAhead>([&](auto m) STEM_INLINE { ring[m] = op[HS + m]; });
            if (mask_from < KT) mask_half(0, mask_from, mask_all);
            if constexpr (!kPastHalf) {
#pragma unroll
                for (int qt = 0; qt < QW; ++qt) {
                    m_ref[qt] = half_max(0, qt, TP);
                    off[qt] = negated_offset(qt);
                }
                note_unseen();
                softmax_pairs(C0{}, C0{}, kHalf{});
            }
        }
        // ---- second half of block `it`, first half of the next ----
#pragma unroll 1
        for (int it = 0; it + 1 < cnt; ++it) {
            if constexpr (kTail) {
                if (((it + 2) & 63) == 0) list_reg = list_chunk(it + 2);
                const int j_then = __builtin_amdgcn_readlane(list_reg, (it + 2) & 63);
                {
                    const auto rk = k_request(clamped(j_nxt));
                    const auto rv = v_request(clamped(j_nxt));
                    phase(C1{}, mask_from, mask_all, [&](int m) STEM_INLINE {
#pragma unroll
                        for (int u = 0; u < KR / 2; ++u) {
                            if (m == 2 * HS - kAhead + u) issue_k(rk, u + KR / 2);
                            if (m == 2 * HS - kAhead + u + KR / 2) issue_v(rv, u);
                        }
                    });
                }
                j_cur = j_nxt;
                j_nxt = j_then;
                block_mask(j_cur, mask_from, mask_all);
                {
                    const auto rk = k_request(clamped(j_nxt), it + 2 < cnt);
                    const auto rv = v_request(clamped(j_cur));
                    phase(C0{}, mask_from, mask_all, [&](int m) STEM_INLINE {
#pragma unroll
                        for (int u = 0; u < KR / 2; ++u) {
                            if (m == 2 * HS - kAhead + u) issue_k(rk, u);
                            if (m == 2 * HS - kAhead + u + KR / 2) issue_v(rv, u + KR / 2);
                        }
                    });
                }
                continue;
            }
            if (((it + 1) & 63) == 0) list_reg = list_chunk(it + 1);
            j_nxt = __builtin_amdgcn_readlane(list_reg, (it + 1) & 63);
            {
                const auto rk = k_request(clamped(j_nxt));
                const auto rv = v_request(clamped(j_cur));
                phase(C1{}, mask_from, mask_all, [&](int m) STEM_INLINE {
#pragma unroll
                    for (int u = 0; u < KR / 2; ++u) {
                        if (m == request_slot(u)) issue_k(rk, u);
                        if (m == request_slot(u + KR / 2)) issue_v(rv, u + KR / 2);
                    }
                });
            }
            j_cur = j_nxt;
            block_mask(j_cur, mask_from, mask_all);
            {
                const auto rk = k_request(clamped(j_cur));
                const auto rv = v_request(clamped(j_cur));
                phase(C0{}, mask_from, mask_all, [&](int m) STEM_INLINE {
#pragma unroll
                    for (int u = 0; u < KR / 2; ++u) {
                        if (m == request_slot(u)) issue_k(rk, u + KR / 2);
                        if (m == request_slot(u + KR / 2)) issue_v(rv, u);
                    }
                });
            }
        }
        // ---- second half of the last block.  On the diagonal block the waves whose queries come before it leave it out of
        //      both products: their neighbours on the SIMD gain.  (Its softmax they make of what lies in the registers and do
        //      not use: a branch around it would have the code of O^T twice.) ----
        const bool second = mask_from == KT || mask_all || w_tile >= TP;
        if constexpr (!kTail) {
            const auto rv = v_request(clamped(j_cur));
#pragma unroll
            for (int u = KR / 2; u < KR; ++u) issue_v(rv, u);
        }
        // (A tile of values whose keys all come after the wave's queries is left out of O^T: a NaN or inf there would not stay
        // out by its weight of zero.)
        const int last_tile = mask_from == KT || mask_all ? KT - 1 : w_tile;
        auto output_half = [&](auto P_tag, auto under) STEM_INLINE {
            constexpr int P = decltype(P_tag)::value;
            u32x4_t op[HS + kAhead];
            unrolled<kAhead>([&](auto m) STEM_INLINE {
                op[m] = load_v(P, m);
                if (m & 1) STEM_SCHED_FENCE();
            });
            auto operand = [&](auto m_tag) STEM_INLINE {
                constexpr int m = decltype(m_tag)::value, a = m + kAhead;
                if constexpr ((m & 1) == 0) {
                    if constexpr (a < HS) {
                        op[a] = load_v(P, a);
                        op[a + 1] = load_v(P, a + 1);
                    }
                    waited(a < HS ? 2 * kAhead : 2 * (HS - m - 2));
                }
                outputs(P_tag, m_tag, op[m & ~1], op[m | 1], [&](auto h) STEM_INLINE {
                    under(std::integral_constant<int, QW * m + decltype(h)::value>{});
                });
            };
            unrolled<KS>(operand);
            if constexpr (TP == 2) {
                if (last_tile > P * TP)
                    unrolled<KS>([&](auto m) STEM_INLINE { operand(std::integral_constant<int, KS + decltype(m)::value>{}); });
            }
            // (where paths meet the compiler may move O to other registers)
            if constexpr (kAcc) wait_states_output<8, kAcc>(o_acc);
        };
        if (second) {
            u32x4_t op[HS + kAhead];
            unrolled<kAhead>([&](auto m) STEM_INLINE { op[m] = ring[m]; });
            unrolled<HS>([&](auto m_tag) STEM_INLINE {
                constexpr int m = decltype(m_tag)::value, a = m + kAhead;
                if constexpr ((m & 1) == 0) {
                    if constexpr (a < HS) {
                        op[a] = load_k(1, a);
                        op[a + 1] = load_k(1, a + 1);
                    }
                    waited(a < HS ? kAhead : HS - m - 2);
                }
                scores(C1{}, m_tag, op[m & ~1], op[m | 1], [&](auto h) STEM_INLINE {
                    softmax_under(C0{}, kHalf{}, kHalf{}, std::integral_constant<int, QW * m + decltype(h)::value>{}, kSpan{});
                });
            });
            if (mask_from < KT) mask_half(1, mask_from, mask_all);
        } else {
            softmax_pairs(C0{}, kHalf{}, kHalf{});
#pragma unroll
            for (int x = 0; x < 2 * QW * TP; ++x) asm volatile("" : "=v"(s_acc[1][x / (2 * QW)][(x / QW) & 1][x % QW]));
        }
        check_half(C0{}, second);
        output_half(C0{}, [&](auto at) STEM_INLINE { softmax_under(C1{}, C0{}, kAll{}, at, kSpan{}); });
        STEM_WAIT_VMCNT(0);
        STEM_BARRIER();                                // the second half of V is there
        if (second) {
            check_half(C1{});
            output_half(C1{}, nothing);
        }
    }
    STEM_WAIT_VMCNT(0);                                // no request may outlive the workgroup's LDS
    wait_states_output<16, kAcc>(o_acc);               // the last O^T instructions have written

    // ---- normalise and store: accumulator x of column tile dt is column dt*16 + 4*(lane/16) + x.  Two column tiles at a time,
    //      one exchange between neighbouring groups of 16 lanes per packed register gives each lane eight consecutive columns,
    //      i.e. 16-byte stores.  (The exchange runs in every lane, valid query or not.) ----
    const int lane_end = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));   // not held through the blocks
    const int c_end = lane_end & 15, g_end = lane_end >> 4;
#pragma unroll
    for (int qt = 0; qt < QW; ++qt) {
        const float inv = l_run[qt] > 0.f ? 1.0f / l_run[qt] : 0.f;
        uint4 packed[KD];
#pragma unroll
        for (int x = 0; x < KD; ++x) {
            const f32x4_t a = o_acc[2 * x][qt], b = o_acc[2 * x + 1][qt];
            const uint32_t a0 = pack_bf16(a[0] * inv, a[1] * inv), a1 = pack_bf16(a[2] * inv, a[3] * inv);
            const uint32_t b0 = pack_bf16(b[0] * inv, b[1] * inv), b1 = pack_bf16(b[2] * inv, b[3] * inv);
            const auto s0 = __builtin_amdgcn_permlane16_swap(a0, b0, false, false);
            const auto s1 = __builtin_amdgcn_permlane16_swap(a1, b1, false, false);
            packed[x] = make_uint4(s0[0], s1[0], s0[1], s1[1]);
        }
        const int tok = row.tok_q0 + (w * QW + qt) * 16 + c_end;
        if (tok < row.q_hi) {
            uint16_t* dst = out + (int64_t)tok * q_st + (int64_t)row.h * q_sh + (g_end & 1) * 16 + (g_end >> 1) * 8;
#pragma unroll
            for (int x = 0; x < KD; ++x) *reinterpret_cast<uint4*>(dst + x * 32) = packed[x];
            if (lse != nullptr && g_end == qt)
                lse[(int64_t)row.h * T + tok] = l_run[qt] > 0.f ? m_ref[qt] * scale + __logf(l_run[qt]) : neg_inf;
        }
    }
}

// QW: 16-query tiles per wave (launch_sparse_attn says when one)
template <int B, int D, int QW>
__global__ __launch_bounds__(B * 4 / QW, D == 256 && QW == 2 ? 1 : 2) void sparse_attn_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    const int32_t* __restrict__ counts, const int32_t* __restrict__ indices,
    uint16_t* __restrict__ out, float* __restrict__ lse, SeqTable seq, RowWalk walk, int Hq, int R, int G,
    int order, int claim_from, int T, int kmax, bool shared_lists, int64_t q_st, int64_t q_sh, int64_t kv_st, int64_t kv_sh,
    float scale, int items_per_xcd, int xcds_per_kv_head, int32_t* __restrict__ taken) {
    __shared__ __attribute__((aligned(1024))) unsigned char lds[4 * B * D];   // the halves of V, then those of K
    unsigned char* k_lds = lds + (kKeysBeyondOffset<B, D> ? 0 : 2 * B * D);
    RowPlace row;
    if (!find_row<B, D != 256>(seq, walk, Hq, R, G, order, claim_from, items_per_xcd, xcds_per_kv_head, taken,
                           reinterpret_cast<int*>(lds), row)) return;
    sparse_attn_body<B, D, QW>(q, k, v, counts, indices, out, lse, row, R, T, kmax, shared_lists, q_st, q_sh, kv_st,
                               kv_sh, scale, k_lds, k_lds + B * D, lds, lds + B * D);
}

int launch_sparse_attn(const Problem& p, const void* q, const void* k, const void* v,
                       const int32_t* counts, const int32_t* indices, int32_t kmax,
                       bool lists_per_kv_head, float softmax_scale, void* out, float* lse,
                       int32_t* queue, hipStream_t stream) {
    // (the host entry point has checked that one sequence of one KV head spans less than 2 GiB: the
    // block requests use a 32-bit byte offset, with offsets from 2^31 on reserved for "fetch nothing")
    const int64_t items = (int64_t)p.Hq * p.R;
    const AttentionGrid ag = attention_grid(p, kmax, queue != nullptr);
    if (ag.slots * 8 > kMaxWorkgroups) return STEM_ERR_UNSUPPORTED;
    dim3 grid((unsigned)(ag.slots * 8));
    // The walk's order is for batches of ten sequences and more, at d = 64 and 128, where rows wait for a place (1.5
    // to 8 times what runs at a time: two workgroups per CU at B = 128, four at B = 64), lists grow with the row
    // (kmax is more than half of the longest sequence's blocks, and these are three or more) and the sequences
    // come in another order.  Attention alone, the walk's order against rows from the last to the first: 149 such batches from
    // 6 % slower to 19 % faster, 6 % in the middle.  Beyond the lines it is worth less or chance prevails: 1.1 to 1.5 times (64
    // batches) 7 % slower to 24 % faster, 7 % in the middle; more than 8 times (66) 1 % slower to 7 % faster, 2 %; two to nine
    // sequences (79) 5 % slower to 19 % faster, 1 %; lists cut to a third and less (68) 4 % slower to 9 % faster, nothing; two blocks at
    // most (74) 10 % slower to 10 % faster, 1 %; d = 256 (with 32 x 32 x 16 products, 23) 5 % slower to 17 % faster, nothing.
    // Batches in ascending order start with the longest as they are and would pay the lookup, up to 5 %.
    RowWalk walk = {};
    int order = p.batch > 1 ? kAsPacked : kOneSequence;
    auto last_block = [&](int s) { return p.seq.first_block[s] + p.seq.row_start[s + 1] - p.seq.row_start[s]; };
    const int64_t at_a_time = p.batch >= 10 && p.d != 256 ? (int64_t)compute_units() * (256 / p.B) : 0;
    if (items * 2 > at_a_time * 3 && items <= at_a_time * 8) {
        bool ascending = true;
        int longest = last_block(0);
        for (int x = 1; x < p.batch; ++x) {
            ascending = ascending && last_block(x - 1) <= last_block(x);
            longest = last_block(x) > longest ? last_block(x) : longest;
        }
        if (!ascending && longest > 2 && kmax > longest / 2) order = kWalk;
    }
    if (order == kWalk) {
        for (int x = 0; x < p.batch; ++x) {            // insertion sort of at most 64
            int y = x;
            for (; y > 0 && last_block(walk.seq[y - 1]) < last_block(x); --y) walk.seq[y] = walk.seq[y - 1];
            walk.seq[y] = (uint8_t)x;
        }
        for (int x = 0, rows = 0; x < STEM_MAX_BATCH; ++x) {
            walk.start[x] = rows;
            if (x < p.batch) rows += p.seq.row_start[walk.seq[x] + 1] - p.seq.row_start[walk.seq[x]];
        }
    }
    const uint16_t* qq = static_cast<const uint16_t*>(q);
    const uint16_t* kk = static_cast<const uint16_t*>(k);
    const uint16_t* vv = static_cast<const uint16_t*>(v);
    uint16_t* oo = static_cast<uint16_t*>(out);
    if (ag.slots > ag.items_per_xcd) hipLaunchKernelGGL(clear_row_queues_kernel, dim3(1), dim3(8), 0, stream, queue);
#define STEM_ATTN_LAUNCH(BB, DD, QW)                                                                        \
    hipLaunchKernelGGL((sparse_attn_kernel<BB, DD, QW>), grid, dim3(BB * 4 / QW), 0, stream, qq, kk, vv, counts, indices, \
                       oo, lse, p.seq, walk, p.Hq, p.R, p.G, order, ag.claim_from, p.T, kmax, lists_per_kv_head, p.q_st, p.q_sh, \
                       p.kv_st, p.kv_sh, softmax_scale, ag.items_per_xcd, ag.xcds_per_kv_head, queue)
    // One 16-query tile per wave, and twice the waves: a CU reads each LDS operand twice as often, and a row takes less time.
    // The better one where the chip has room for the waves, where rows of different length leave the longest to run by themselves
    // (`grow`: from the start of prompts, with lists of more than half of their blocks), and where lists are short.  The bits are the
    // same.  One tile / two, attention alone, 1 to 150 blocks per list, whole and packed prompts and late chunks of long ones:
    //   B = 128, d = 128: up to a row per CU 0.88 to 1.04; up to two, grow 0.84 to 0.99, else 0.95 to 1.33, grow in batches 0.94 to 1.21.
    //     d = 64: up to a row per CU 0.83 to 1.00; up to two, grow 0.85 to 1.00, else 0.87 to 1.08.
    //   B = 64: up to two rows per CU, d = 128 0.74 to 1.04, d = 64 0.75 to 1.05; up to three with 12 to 80 blocks 0.79 to 1.00 and, at
    //     d = 64, with more 0.89 to 0.98; with fewer 0.83 to 1.23, but at d = 64 and up to 2 3/4 rows 0.81 to 0.99; up to four, grow
    //     0.82 to 1.04, else 0.82 to 1.30.
    //   d = 256, B = 64: up to a row per CU 0.72 to 0.98; up to three of at most 50 blocks, or grow, 0.72 to 1.03, of more 0.88 to
    //     1.27; up to six of at most 20 and 16 of at most 10 0.67 to 1.02, beyond 0.87 to 1.17.  B = 128: of 4 blocks 0.91 to 1.01,
    //     of 8 0.98 to 1.04, of 12 1.00 to 1.06, of 100 1.04 to 1.11.
    const int64_t cus = compute_units();
    const bool grow = (p.batch == 1 || p.B == 64 || p.d == 64) && 4 * (int64_t)p.R >= 3 * (int64_t)p.NBmax && 2 * (int64_t)kmax > p.NBmax;
    const bool narrow =
        p.d == 256 && p.B == 128 ? items <= 16 * cus && kmax <= 8
        : p.d == 256 ? items <= cus || (items <= 3 * cus && (kmax <= 50 || grow)) || (items <= 6 * cus && kmax <= 20) ||
                           (items <= 16 * cus && kmax <= 10)
        : p.B == 128 ? items <= cus || (items <= 2 * cus && grow)
                     : items <= 2 * cus || (p.d == 64 && 4 * items <= 11 * cus) ||
                           ((p.d == 64 || kmax <= 80) && ((items <= 3 * cus && kmax >= 12) || (items <= 4 * cus && grow)));
    if (p.B == 128 && p.d == 128 && narrow) STEM_ATTN_LAUNCH(128, 128, 1);
    else if (p.B == 128 && p.d == 128) STEM_ATTN_LAUNCH(128, 128, 2);
    else if (p.B == 64 && p.d == 128 && narrow) STEM_ATTN_LAUNCH(64, 128, 1);
    else if (p.B == 64 && p.d == 128) STEM_ATTN_LAUNCH(64, 128, 2);
    else if (p.B == 128 && p.d == 64 && narrow) STEM_ATTN_LAUNCH(128, 64, 1);
    else if (p.B == 128 && p.d == 64) STEM_ATTN_LAUNCH(128, 64, 2);
    else if (p.B == 64 && p.d == 64 && narrow) STEM_ATTN_LAUNCH(64, 64, 1);
    else if (p.B == 64 && p.d == 64) STEM_ATTN_LAUNCH(64, 64, 2);
    else if (p.B == 128 && p.d == 256 && narrow) STEM_ATTN_LAUNCH(128, 256, 1);
    else if (p.B == 128 && p.d == 256) STEM_ATTN_LAUNCH(128, 256, 2);
    else if (p.B == 64 && p.d == 256 && narrow) STEM_ATTN_LAUNCH(64, 256, 1);
    else if (p.B == 64 && p.d == 256) STEM_ATTN_LAUNCH(64, 256, 2);
    else return STEM_ERR_UNSUPPORTED;
#undef STEM_ATTN_LAUNCH
    return check_launch();
}

}  // namespace stem
