// Internal helpers shared by the translation units of libmoe_janus (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>

#include "moe_janus.h"

#define MOE_WAVE 64

struct moe_placement {
    int E, n_inst, C;
    int n_words;                 // ceil(E/64): 64-bit words of an expert bitset
    // host tables
    int32_t *slot_to_expert_h;   // [n_inst*C]
    int32_t *R_h;                // [E]
    // device tables (one allocation, 256-byte aligned sub-arrays)
    void     *dev_block;
    uint64_t *host_mask_d;       // [E]  bit g set <=> instance g hosts a replica of e
    int16_t  *slot_of_d;         // [E*n_inst] local slot of e on g, -1 if not hosted
    int32_t  *single_rid_d;      // [E]  RID when R(e) == 1, else -1
    uint64_t *multi_mask_d;      // [n_words] bit e set <=> R(e) > 1
    uint64_t *single_mask_d;     // [n_inst*n_words] single-replica experts hosted on g
    int device;
};

namespace moe {

void set_hip_error(hipError_t e, const char *where);

inline int check_launch(const char *where) {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        set_hip_error(e, where);
        return MOE_EHIP;
    }
    return MOE_OK;
}

// Control region at the start of the FFN workspace: a header of 256 ints, then the hand-off counters
// of the blocks (ffn_stream.hip).  Header words: the status bits, and the per-workspace options
// that moe_workspace_set_option writes and moe_workspace_init resets to 0 (= the default).
constexpr size_t kFfnCtrlBytes = 4u << 20;
constexpr int kCtrlStatus = 1;           // bit 0: a wait overran; bit 1: list cut for another block size
constexpr int kCtrlSpinLimit = 2;        // polls a stage-2 workgroup spends on a block's flag before it gives up
constexpr int kCtrlWideMin = 3;          // workgroups of wide blocks a batch must have for them to be used (ffn_stream.hip)

// Blocks of the work list that get workgroups of their own in the streaming launch (longer lists wrap around)
constexpr unsigned kFfnLaneBlocks = 128;

// Request rows per block of the FFN work list: small batches take blocks of 32 rows (more, shorter
// workgroups), larger ones blocks of 64 (hot slots then re-read their expert half as often).
inline int ffn_block_rows(int T) { return T < 384 ? 32 : MOE_FFN_BLOCK_ROWS; }

// Upper bound of the number of blocks over all slots, whatever the requests are (also when a
// token names one expert several times): every slot has at most one partly filled block, and
// the full ones hold T*k requests at most.
inline long long ffn_max_blocks(int T, int k, int C) {
    return C + static_cast<long long>(T) * k / ffn_block_rows(T);
}

// Bytes of the intermediate `act` per entry of the work list: a block of rows x d_e rounded up to
// whole 128-byte lines (64 channels).  A wide block (ffn_stream.hip) uses the regions of the entries
// it spans.
inline size_t ffn_act_block_bytes(int T, int d_e) {
    return static_cast<size_t>(ffn_block_rows(T)) * ((d_e + 63) / 64 * 64) * 2;
}
inline size_t ffn_stream_act_bytes(int T, int k, int C, int d_e) {
    const size_t b = static_cast<size_t>(ffn_max_blocks(T, k, C)) * ffn_act_block_bytes(T, d_e);
    return (b + 255) / 256 * 256;
}

// One set of experts of a bf16 grouped FFN: C slots of width d_e, k requests a token.
struct FfnCall {
    const void *X, *W13p, *W2p;
    int k, C, d_e;
    const int32_t *blocks, *perm;
    int *ctrl;                           // the workspace's control region
    uint16_t *act;                       // ffn_stream_act_bytes(T, k, C, d_e) bytes
    float *Yp;
};

// bf16 grouped FFN (ffn_stream.hip); shapes validated by the caller.  `ctrl` is the zero-initialised
// control region of the workspace.  Returns MOE_OK or MOE_ESHAPE (too many blocks).
int launch_ffn_stream(const FfnCall &c, int T, int d_h, hipStream_t st);
// The same for two sets of experts over the same token rows in one launch, where ffn_stream_takes_shared() says so.
bool ffn_stream_takes_shared(const FfnCall &c, const FfnCall &sh, int T, int d_h);
void launch_ffn_stream_shared(const FfnCall &c, const FfnCall &sh, int T, int d_h, hipStream_t st);

// Batches that take the launch for large batches (ffn_big_kernel; block lists of 64 rows): from 2048 tokens on, and below
// where T x d_h x d_e is large, unless the slots have few requests even if all of them are local.  Us a layer in that launch and in the
// streaming launch: T = 2040, d_h = 4096, d_e = 1536 170 and 197; T = 1000, d_h = 7168, d_e = 2048 275 and 276, T = 2040 356 and 362;
// but T = 1000, d_h = 4096, d_e = 1536 155 and 152; d_h = 2048, d_e = 1408 97 and 89; T = 2000 120 and 114.  From 2048 tokens on it is the
// faster one where the batch has many wide blocks, which the host cannot know (64 slots of 250 rows, d_h = 1024, d_e = 512 102 and 131;
// T = 8000, d_h = 2048, d_e = 768, zipf 1 126 and 157); but 64 to 131 requests a slot, of which a quarter is local, 3-12 % slower.
// At most 56 requests a slot on average leave few slots with more than 64, and streaming items want the third workgroup a CU: 200
// slots of 20 rows, d_h = 512, d_e = 256 57 and 42; 100 of 50, d_h = 1024, d_e = 512 94 and 79; popular slots of
// up to 400 rows cost at most 5 % (160 slots, 52 on average, zipf 0.6, d_h = 7168, d_e = 256 516 and 545).  With 63 on average, all
// local, half of the slots are wide: 132 slots, d_h = 4096, d_e = 1536 1028 and 1201.
constexpr int kBigMinTokens = 2048;
constexpr long long kBigWork = 12000000000LL;
constexpr int kBigMinRows = 56;
inline bool ffn_is_big(int T, int k, int C, int d_h, int d_e) {
    if (static_cast<long long>(T) * k <= static_cast<long long>(kBigMinRows) * C) return false;
    return T >= kBigMinTokens || (ffn_block_rows(T) == 64 && static_cast<long long>(d_h) * d_e >= kBigWork / T);
}

inline bool aligned(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

__device__ __forceinline__ int lane_id() { return threadIdx.x & (MOE_WAVE - 1); }

__device__ __forceinline__ uint64_t lanemask_lt() {
    return (1ull << lane_id()) - 1ull;
}

__device__ __forceinline__ float bf16_to_f32(uint16_t b) {
    return __uint_as_float(static_cast<uint32_t>(b) << 16);
}

// Two values as bf16, round-to-nearest-even, NaN stays NaN: v_cvt_pk_bf16_f32, lo in the low half.
__device__ __forceinline__ uint32_t f32x2_to_bf16x2(float lo, float hi) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{lo, hi}), bf16x2));
}

// round-to-nearest-even; NaN stays NaN
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return static_cast<uint16_t>((u >> 16) | 0x40u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return static_cast<uint16_t>(u >> 16);
}

}  // namespace moe
