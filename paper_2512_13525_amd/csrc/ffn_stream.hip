// a5, bf16 path: the grouped expert FFN (gate/up + SiLU*up, then down) as oversubscribed streaming
// workgroups.
//
// Janus Sec. 2.2: at decode sizes an expert is two skinny GEMMs whose cost is the weight bytes
// streamed from HBM, so the layer's latency follows the number of activated experts.  The work
// of a stage is cut into items = (block of up to 32 or 64 request rows of one slot) x (tile of 16
// gate+up channels in stage 1, 32 output channels in stage 2); one workgroup per item, in plain
// grid order, dispatched by the hardware.  Slots without requests own no item: their weights are
// never read.  Nothing about the activated set is known on the host, so the grid is sized for
// the largest possible number of blocks; the dispatch step leaves the list of blocks in device
// memory, a workgroup reads its entry with two scalar loads, and workgroups past the last block
// leave at once.
//
// The 4 wavefronts of a workgroup split the K dimension of the tile round-robin in super-steps
// of 64 columns and meet in LDS once, at the end (fixed summation order: results are
// reproducible).  Per super-step a wavefront reads 4 KiB of weights (packed MFMA A-operand
// images, fully coalesced 128-bit loads, two super-steps ahead) and the token rows (the B operand,
// from L2).  In stage 1 those are gathered rows of X: one 128-byte line of each row, one super-step
// ahead, turned into the MFMA layout through a wave-private LDS tile.  Stage 1 writes `act` as
// B-operand images, so stage 2 reads its token fragments like the weights, straight into
// registers and as far ahead.
//
// Every further streaming block of a slot streams the expert's tiles again.  When a batch has enough
// slots with more than 64 requests (wide_on below), those slots are computed as tiled GEMMs over
// blocks of 64 rows by workgroups of the same launch instead (wide_item): a workgroup takes four
// channel tiles through the whole K dimension, shares the token rows of the block between them
// through LDS, and the blocks of a slot are dealt to the workgroups so that they find the
// expert's tiles in their XCD's L2 (run_wide).  Large batches have a launch of their own kind
// (ffn_big_kernel): the same two stages and hand-off, larger wide blocks first, streaming items for the rest.
//
// Both stages run in ONE launch: the stage-2 workgroups have the higher ids, so the hardware
// starts them only after every stage-1 workgroup has been started, and they fill the compute
// units that the tail of stage 1 leaves idle.  A streaming workgroup of stage 2 first puts its weight loads
// in flight (a tiled-GEMM one requests nothing yet) and then waits until the 16-channel tiles of its block of `act` rows are all written: a
// counter per block in the workspace is bumped by each stage-1 workgroup once its stores are
// acknowledged; the workgroup that completes the count raises the block's ready flags, which the
// stage-2 workgroups poll (bounded; on an overrun the workgroup raises the workspace's error word,
// writes NaN rows instead of results and leaves, so every wave reaches the end of the kernel).  The 8 XCDs do not share an
// L2: `act` is written with agent-scope (write-through) stores, every 128-byte line of it has one
// writing workgroup, and no workgroup reads a line before its block is ready, so plain loads see
// the data; counters and flags are agent-scope atomics.  The last stage-2 workgroup of a block to
// get through the wait clears the block's control lines for the next call.
#include "dispatch_dev.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kDepthA = 2;              // super-steps of weight loads each wavefront keeps in flight
constexpr int kThreads = 256;
constexpr int kWaves = kThreads / MOE_WAVE;
// A launch is compiled for blocks of TT token tiles of 16 rows (TT = 2 or 4: blocks of 32 or 64
// request rows); one 16-channel tile of a block of act takes TT*16 rows x 32 bytes.

// Control region of the workspace (ints): [1] error word; block j owns the 8 lines of 128 bytes
// at int offset (j+1)*kCtrlBlockInts: line 0 = {stage-1 tiles done, stage-2 workgroups through},
// lines 1..7 = copies of the block's ready flag (same-address accesses from many workgroups
// serialise in the memory system, so the pollers are spread over the copies).
constexpr int kCtrlLineInts = 32;
constexpr int kCtrlCopies = 7;
constexpr int kCtrlBlockInts = (1 + kCtrlCopies) * kCtrlLineInts;
constexpr int kMaxItems = static_cast<int>(moe::kFfnCtrlBytes / 4) / kCtrlBlockInts - 1;

// Division of 0 <= x < 2^31 by a divisor that the host knows: x / d = (2x * mul) >> (32 + shift), exact with
// mul = ceil(2^(31 + shift) / d) and 2^shift >= d (the excess mul * d - 2^(31 + shift) stays below d <= 2^shift, so it adds
// less than 1 / d to the quotient).
struct FastDiv {
    uint32_t mul;
    int shift;
    __device__ __forceinline__ uint32_t operator()(uint32_t x) const { return __umulhi(x << 1, mul) >> shift; }
};

FastDiv fast_div(uint32_t d) {
    FastDiv f{0, 0};
    while ((1ull << f.shift) < d) ++f.shift;
    f.mul = static_cast<uint32_t>(((1ull << (31 + f.shift)) + d - 1) / d);
    return f;
}

struct StageArgs {
    const uint16_t *B;                   // token operand: X (stage 1, rows through perm) or act (stage 2, blocks)
    const char *Wp;                      // packed weights: [C][tiles][KS][2][64] fragments of 16 bytes
    int tiles, items, tiles_pad, KS;     // items = workgroups per block (stage 2: one per pair of tiles); tiles_pad = items rounded up to a multiple of 8
    FastDiv pad_div;                     // division by tiles_pad
    int b_stride;                        // elements between rows of X (stage 1)
    int out_stride;                      // elements between rows of Yp (stage 2)
};

struct StreamArgs {
    StageArgs s[2];
    const int32_t *blocks;               // work list written by the dispatch step
    const int32_t *perm;
    uint16_t *act;                       // stage-1 output
    float *Yp;                           // stage-2 output
    int *ctrl;
    FastDiv k_div;                       // division by k: token of a request
    int spin_limit;
    unsigned list_last;                  // index of the last entry the work list has room for
    uint32_t act_block_bytes;            // bytes of `act` per entry of the work list: R rows x d_e rounded up to 64 channels
};

// The work list and the header of the control region do not change while the launch runs: read through the constant address
// space, they are scalar loads that the compiler may issue together, ahead of everything else.  (As plain loads they were
// vector loads behind the stores and atomics of the kernel, four dependent round trips before a workgroup's first operand.)
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ int4 load_const(const int32_t *p, unsigned i) {
    const i32x4 v = reinterpret_cast<const __attribute__((address_space(4))) i32x4 *>(reinterpret_cast<uintptr_t>(p))[i];
    return make_int4(v[0], v[1], v[2], v[3]);
}

__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// The weights of a slot with a single block are read exactly once: they are loaded with the
// streaming hint (STREAM), so that on their way through an L2 they do not push out the token rows,
// which every tile of a block reads again (7 MB of rows against a 4 MB L2 at d_h = 7168, T = 512:
// 237 -> 227 us for that launch).  The blocks of a slot with several share their tiles through L2
// and keep the plain loads, the last, partly filled one too (with the hint on those all-slot batches of 128 to 512 tokens
// were 20 % slower; with it on the last block alone, slots of 36 to 60 rows at d_h = 2048, d_e = 768 43 us, 33 without,
// 47.7 and 42.6 with the weights out of the caches).
template <bool STREAM>
__device__ __forceinline__ bf16x8 load_weights(const char *p) {
    if constexpr (STREAM) return __builtin_nontemporal_load(reinterpret_cast<const bf16x8 *>(p));
    else return *reinterpret_cast<const bf16x8 *>(p);
}

__device__ __forceinline__ float silu_mul(float g, float u) { return g / (1.0f + __expf(-g)) * u; }

// Waits until at most N of this wavefront's loads are outstanding.
template <int N>
__device__ __forceinline__ void wait_loads() {
    __builtin_amdgcn_s_waitcnt((N & 15) | (N >> 4) << 14 | 7 << 4 | 15 << 8);
}

// Workgroup barrier for LDS exchange only: waits for this wavefront's LDS traffic, not for its
// global loads (prefetched weights stay in flight across it).
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Partial sums of an item in LDS: [wave][fragment][lane] (a fragment = 16 channels x 16 rows), at most 2*TT fragments.
// F fragments of NT row tiles each are stored fragment-major: f * NT + t.
template <int F, int NT, int TT>
__device__ __forceinline__ void put_partials(char *lds, const f32x4 (&acc)[F][NT], int wave, int lane) {
    static_assert(F * NT <= 2 * TT, "the reduction buffer holds 2 * TT fragments per wavefront");
    f32x4 *red = reinterpret_cast<f32x4 *>(lds) + wave * (2 * TT * MOE_WAVE) + lane;
#pragma unroll
    for (int f = 0; f < F; ++f)
#pragma unroll
        for (int t = 0; t < NT; ++t) red[(f * NT + t) * MOE_WAVE] = acc[f][t];
}

template <int TT>
__device__ __forceinline__ f32x4 sum_partials4(const char *lds, int frag, int lane) {
    const f32x4 *red = reinterpret_cast<const f32x4 *>(lds) + frag * MOE_WAVE + lane;
    f32x4 v = red[0];
#pragma unroll
    for (int wv = 1; wv < kWaves; ++wv) v += red[wv * (2 * TT * MOE_WAVE)];
    return v;
}

// One value of a fragment's 256 (value v: lane v / 4, element v % 4).
template <int TT>
__device__ __forceinline__ float sum_partials(const char *lds, int frag, int v) {
    const float *red = reinterpret_cast<const float *>(lds) + frag * (4 * MOE_WAVE) + v;
    float s = red[0];
#pragma unroll
    for (int wv = 1; wv < kWaves; ++wv) s += red[wv * (2 * TT * MOE_WAVE * 4)];
    return s;
}

// The value of another lane of the same four.
template <int A, int B, int C, int D>
__device__ __forceinline__ uint32_t quad_perm(uint32_t v) {
    return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), A | B << 2 | C << 4 | D << 6, 0xf, 0xf, false));
}
template <int A, int B, int C, int D>
__device__ __forceinline__ float quad_perm(float v) { return __uint_as_float(quad_perm<A, B, C, D>(__float_as_uint(v))); }

// Split-K reduction over the 4 wavefronts in LDS (fixed order), then the epilogue: SiLU(gate)*up
// rounded once to bf16 (stage 1, agent-scope stores) or the fp32 partial output rows (stage 2).  One copy of this code
// for all numbers of row tiles (nt): the kernel's instructions are many times the instruction cache.
template <int TT>
__device__ __forceinline__ void store_act(const StreamArgs &a, const char *lds, int nt, int item_id, int tile, int row0, int row_end) {
    // Value v of a fragment (v / 4 = lane l, v % 4 = i) is gate/up channel tile*16 + (l/16)*4 + i of token row0 + t*16 + l%16: a
    // thread takes one value of each row tile, so that all wavefronts share the work however few the rows are (with four
    // values a thread a block of up to 16 rows was one wavefront's, 0.7 us of a chain that stage 2 waits for: four layer
    // steps with five blocks of up to 5 rows 92.2 -> 91.0 us, with 12 of up to 32 rows 114.3 -> 112.9).
    const int l = threadIdx.x >> 2, i = threadIdx.x & 3;
    // act block of this item: [K-step of stage 2][token tile][64 lanes][16 B], the register image of
    // the MFMA B operand (lane: row % 16, channels (lane / 16) * 8 .. + 7 of the K-step's 32); this
    // tile is half a K-step, and every 128-byte line of the image has one writing workgroup
    const int fl = (l & 15) + 16 * ((tile & 1) * 2 + (l >> 5));
    char *dst = reinterpret_cast<char *>(a.act) + static_cast<size_t>(item_id) * a.act_block_bytes +
                static_cast<size_t>(tile >> 1) * (TT * 1024) + fl * 16 + ((l >> 4) & 1) * 8;
#pragma unroll 1
    for (int t = 0; t < nt; ++t) {
        const float act = silu_mul(sum_partials<TT>(lds, t, threadIdx.x), sum_partials<TT>(lds, nt + t, threadIdx.x));
        // the four channels of a quad of threads, stored by its first
        const uint32_t hi = moe::f32x2_to_bf16x2(act, quad_perm<1, 1, 3, 3>(act));   // lanes 0 and 2 of the quad: channels i, i+1
        const uint64_t o = hi | static_cast<uint64_t>(quad_perm<2, 2, 2, 2>(hi)) << 32;
        if (i == 0 && row0 + t * 16 + (l & 15) < row_end)
            __hip_atomic_store(reinterpret_cast<uint64_t *>(dst + t * 1024), o, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// nf fragments of 16 output channels, from channel tile*32 on
template <int TT>
__device__ __forceinline__ void store_rows(const StreamArgs &a, const StageArgs &g, const char *lds, int nf, int nt, int tile,
                                           int row0, int row_end) {
    // lane-slot (f, t, l) holds output channels tile*32 + f*16 + (l/16)*4 .. +3
    int f = 0, t = threadIdx.x / MOE_WAVE;
    for (int item = threadIdx.x; item < nf * nt * MOE_WAVE; item += kThreads, t += kWaves) {
        while (t >= nt) { t -= nt; ++f; }
        const int l = item % MOE_WAVE;
        const f32x4 y = sum_partials4<TT>(lds, item / MOE_WAVE, l);
        const int r = row0 + t * 16 + (l & 15);
        if (r < row_end)
            *reinterpret_cast<f32x4 *>(a.Yp + static_cast<size_t>(r) * g.out_stride + tile * 32 + f * 16 + (l >> 4) * 4) = y;
    }
}

// Stage 2 of a block may read `act` only when all stage-1 tiles of the block are written: the
// stage-1 workgroup that completes the count raises the block's ready flags.  Called by the whole
// workgroup; thread 0 polls one copy of the flag.  The second counter of the block counts the
// stage-2 workgroups that got through: the last one clears the block's control lines for the
// next call.  Returns false when the bounded wait ran out: the status word gets bit 0, the
// block's control lines are left as they are (a late stage-1 tile may still bump them, so the
// region needs moe_workspace_init before the next call), and the caller must not read `act`.
__device__ __forceinline__ bool wait_block_ready(const StreamArgs &a, int *s_ok, int item, int tile, int n_readers) {
    if (threadIdx.x == 0) {
        int *blk = a.ctrl + (item + 1) * kCtrlBlockInts;
        const int *flag = blk + (1 + tile % kCtrlCopies) * kCtrlLineInts;
        // header word 2: a spin limit for this workspace (tests of the overrun path); 0 = the default
        const int lim_ws = load_const(a.ctrl, 0).z;
        const int limit = lim_ws > 0 ? lim_ws : a.spin_limit;
        int spins = 0, ok = 1;
        while (__hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0) {
            if (++spins > limit) {
                __hip_atomic_fetch_or(a.ctrl + moe::kCtrlStatus, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                ok = 0;
                break;
            }
            __builtin_amdgcn_s_sleep(8);
        }
        if (ok && __hip_atomic_fetch_add(blk + 1, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n_readers - 1) {
            __hip_atomic_store(blk, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(blk + 1, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
            for (int c = 1; c <= kCtrlCopies; ++c)
                __hip_atomic_store(blk + c * kCtrlLineInts, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        *s_ok = ok;
    }
    lds_barrier();
    return *s_ok != 0;
}

// A stage-1 workgroup announces its part of a block (one of n): every thread waits for its own act stores to be
// acknowledged, then one thread bumps the block's counter and, if it completes the count, raises the ready flags (every other
// part's stores were acknowledged before its bump).
__device__ __forceinline__ void announce_tiles(const StreamArgs &a, int item, int n) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
        int *blk = a.ctrl + (item + 1) * kCtrlBlockInts;
        if (__hip_atomic_fetch_add(blk, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n - 1) {
#pragma unroll
            for (int c = 1; c <= kCtrlCopies; ++c)
                __hip_atomic_store(blk + c * kCtrlLineInts, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// The rows of a stage-2 item whose block never became ready: quiet NaNs, so that the combine
// propagates them and nobody mistakes the rows for results.
__device__ __forceinline__ void store_nan_rows(const StreamArgs &a, const StageArgs &g, int tile, int row0, int n_rows) {
    const float qnan = __uint_as_float(0x7fc00000u);
    const f32x4 v = {qnan, qnan, qnan, qnan};
    for (int i = threadIdx.x; i < n_rows * 8; i += kThreads)
        *reinterpret_cast<f32x4 *>(a.Yp + static_cast<size_t>(row0 + i / 8) * g.out_stride + tile * 32 + (i % 8) * 4) = v;
}

// One stage-1 item.  A super-step is two K-steps = 64 columns = one 128-byte line of every token row (with an odd
// number of K-steps, hidden sizes that are multiples of 32 but not of 64, two halves of one for every other row: still a
// quarter of the requests of reading 16 bytes per lane straight into the MFMA layout: 52 -> 46 us for the launch at
// d_h = 2016, d_e = 1056, T = 203; a layer whose weights stay in the last-level cache loses at 16 to 32 rows a slot, 36 -> 39).
// A token load instruction fetches whole lines (lane l: row l/8, 16-byte chunk l%8), so no line
// is requested twice and none by halves; the MFMA layout (lane l: row l%16, 16-byte chunk 4*step + l/16) is produced by a
// round trip through a wave-private 2 KiB LDS tile per 16 rows (chunks XOR-swizzled by row so
// that both the row-major writes and the column-wise reads spread over the banks).  NH = number
// of 8-row halves that hold requests (rows past the end repeat the last row; halves past it are
// not loaded and leave unspecified values in token columns whose results are never stored).
// EVEN: the number of K-steps is even.  Otherwise one wavefront adds the last K-step after its super-steps.
template <int NH, int TT, bool STREAM, bool EVEN>
__device__ __forceinline__ void stream_item_lines(const StreamArgs &a, const StageArgs &g, char *lds,
                                                  const char *w, int tile, int row0, int row_end,
                                                  int wave, int lane) {
    asm volatile("" : "+v"(lane));                             // see wide_item
    constexpr int NT = (NH + 1) / 2;
    constexpr int D = kDepthA;
    char *stg = lds + wave * (TT * 2048);
    const uint32_t aoff = lane * 16;
    // token rows: wave-uniform base (advanced per super-step) + constant 32-bit per-lane byte offset
    uint32_t boff[NH];
#pragma unroll
    for (int h = 0; h < NH; ++h) {
        int r = row0 + h * 8 + (lane >> 3);
        r = r < row_end ? r : row_end - 1;
        boff[h] = static_cast<uint32_t>(a.perm[r]);                  // the request; its row's offset below
    }
    asm volatile("" ::: "memory");
    // LDS: row R of a tile at R*128, its 16-byte chunk c at ((c ^ ((R >> 1) & 7)) * 16): the 16 rows a
    // fragment read touches fall into 16 different bank groups.  wr_lds[p]: rows of an even / odd half.
    const uint32_t wr_lds[2] = {static_cast<uint32_t>(((lane >> 3) * 128) + (((lane & 7) ^ (lane >> 4)) * 16)),
                                static_cast<uint32_t>(((lane >> 3) * 128) + (((lane & 7) ^ (4 + (lane >> 4))) * 16))};
    const uint32_t rd_row = (lane & 15) * 128, rd_sw = (lane >> 1) & 7, rd_g = lane >> 4;
    const char *bbase = reinterpret_cast<const char *>(g.B);
    constexpr int kBStep = 128;                                  // bytes a super-step advances a token row
    const int n = (g.KS / 2 - wave + kWaves - 1) / kWaves;      // super-steps wave, wave+4, ... of this wavefront
    f32x4 acc[2][NT];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[h][t] = f32x4{0.f, 0.f, 0.f, 0.f};

    // Weights run D super-steps ahead (ring wr); the token rows DB super-steps: the loads of
    // super-step q+DB are issued in iteration q *before* the weights of q+D.  Loads return in order,
    // so waiting for the token rows of the next super-step also waits for every older weight load.
    // At the top of the loop the compiler allows for the way into it, where the first weights are in front of the first
    // token rows: every D-th super-step waits until nothing or (DB = 1) the rows of one are in flight.  Waiting for the first rows
    // ahead of the loop instead, so that 4 to 16 loads stay in flight, is level or slower (four layer steps with five blocks of up
    // to 5 rows 91.4 and 92.3 us, with 17 of up to 32 rows 154.0 and 155.7; d_h = 7168, T = 512 222.2 and 223.6).
    // Before and after the loop loads are only issued for super-steps that exist.
    constexpr int DB = (NH <= 4) ? D : 1;                        // D: the two rings share their positions
    bf16x8 wr[D][2][2];
    bf16x8 br[DB][NH];
    const int last = n > 0 ? n - 1 : 0;
    // Workgroups start their K loop at different places (and wrap around) so that they do not
    // march through equally aligned tiles in lockstep.
    const int rot = n > 0 ? static_cast<int>(static_cast<unsigned>(tile) % static_cast<unsigned>(n)) : 0;
#define MOE_STEP_INDEX(step)                                                                     \
        const int q_ = (step);                                                                   \
        int r_ = (q_ < last ? q_ : last) + rot;                                                  \
        r_ = r_ >= n ? r_ - n : r_;                                                              \
        const int s_ = wave + kWaves * r_;
#define MOE_LOAD_A(d, step)                                                                      \
    do {                                                                                         \
        MOE_STEP_INDEX(step)                                                                     \
        const char *ws_ = w + static_cast<size_t>(s_) * 4096;                                    \
        _Pragma("unroll") for (int ss = 0; ss < 2; ++ss) {                                       \
            wr[d][ss][0] = load_weights<STREAM>(ws_ + ss * 2048 + aoff);                        \
            wr[d][ss][1] = load_weights<STREAM>(ws_ + ss * 2048 + 1024 + aoff);                 \
        }                                                                                        \
        asm volatile("" ::: "memory");                                                           \
    } while (0)
#define MOE_LOAD_B(d, step)                                                                      \
    do {                                                                                         \
        MOE_STEP_INDEX(step)                                                                     \
        const char *bs_ = bbase + static_cast<size_t>(s_) * kBStep;                              \
        _Pragma("unroll") for (int h = 0; h < NH; ++h)                                           \
            br[(d) % DB][h] = *reinterpret_cast<const bf16x8 *>(bs_ + boff[h]);                  \
        asm volatile("" ::: "memory");                                                           \
    } while (0)
#define MOE_STAGE_B(d)                                                                           \
    do {                                                                                         \
        _Pragma("unroll") for (int h = 0; h < NH; ++h)                                           \
            *reinterpret_cast<bf16x8 *>(stg + (h / 2) * 2048 + (h % 2) * 1024 + wr_lds[h % 2]) = br[(d) % DB][h]; \
        asm volatile("" ::: "memory");                                                           \
    } while (0)
#define MOE_MMA_STEP(d)                                                                          \
    do {                                                                                         \
        _Pragma("unroll") for (int ss = 0; ss < 2; ++ss)                                         \
            _Pragma("unroll") for (int t = 0; t < NT; ++t) {                                     \
                const bf16x8 bf_ = *reinterpret_cast<const bf16x8 *>(                            \
                    stg + t * 2048 + rd_row + (((4 * ss + rd_g) ^ rd_sw) * 16));                 \
                acc[0][t] = mfma16(wr[d][ss][0], bf_, acc[0][t]);                                \
                acc[1][t] = mfma16(wr[d][ss][1], bf_, acc[1][t]);                                \
            }                                                                                    \
        asm volatile("" ::: "memory");                                                           \
    } while (0)
    // The last K-step of an odd number, by the wavefront that is next in turn: its operands are requested before that
    // wavefront's last super-steps are multiplied, the token rows 16 bytes a lane in the MFMA layout (the row offsets
    // come from the lanes that hold them for the whole-line loads).
    const bool extra = !EVEN && wave == (g.KS >> 1) % kWaves;
    bf16x8 xw[2], xb[NT];
#define MOE_LOAD_EXTRA()                                                                         \
    do {                                                                                         \
        if (extra) {                                                                             \
            const char *ws_ = w + static_cast<size_t>(g.KS - 1) * 2048 + aoff;                   \
            xw[0] = load_weights<STREAM>(ws_);                                                   \
            xw[1] = load_weights<STREAM>(ws_ + 1024);                                            \
            _Pragma("unroll") for (int t = 0; t < NT; ++t) {                                     \
                const uint32_t o0_ = __shfl(boff[2 * t], (lane & 7) * 8);                        \
                const uint32_t o1_ = 2 * t + 1 < NH ? __shfl(boff[2 * t + 1 < NH ? 2 * t + 1 : 0], (lane & 7) * 8) : o0_; \
                xb[t] = *reinterpret_cast<const bf16x8 *>(bbase + static_cast<size_t>(g.KS - 1) * 64 + (lane >> 4) * 16 + \
                                                          ((lane & 8) ? o1_ : o0_));             \
            }                                                                                    \
        }                                                                                        \
        asm volatile("" ::: "memory");                                                           \
    } while (0)
    // issue order of the first loads: the weights do not wait for the requests' tokens to be known
#pragma unroll
    for (int d = 0; d < D; ++d)
        if (d < n) MOE_LOAD_A(d, d);
#pragma unroll
    for (int h = 0; h < NH; ++h)
        boff[h] = a.k_div(boff[h]) * static_cast<uint32_t>(g.b_stride) * 2 + (lane & 7) * 16;
    if (n > 0) {
#pragma unroll
        for (int d = 0; d < DB; ++d)
            if (d < n) MOE_LOAD_B(d, d);
        int i = 0;
        for (; i + 2 * D <= n; i += D) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                MOE_STAGE_B(d);
                MOE_LOAD_B(d + DB, i + d + DB);
                MOE_MMA_STEP(d);
                MOE_LOAD_A(d, i + d + D);
            }
        }
        if constexpr (!EVEN) MOE_LOAD_EXTRA();
        const int rem = n - i;                                   // 1 .. 2*D-1 super-steps left
        // the last 1 .. 2*D-1 super-steps: only those that exist are loaded, staged and multiplied
        // (wave-uniform conditions)
#pragma unroll
        for (int d = 0; d < D; ++d) {
            if (d < rem) MOE_STAGE_B(d);
            if (d + DB < rem) MOE_LOAD_B(d + DB, i + d + DB);
            if (d < rem) MOE_MMA_STEP(d);
            if (d < D - 1 && d + D < rem) MOE_LOAD_A(d, i + d + D);
        }
#pragma unroll
        for (int d = 0; d < D - 1; ++d) {
            if (D + d < rem) {
                MOE_STAGE_B(D + d);
                MOE_MMA_STEP(d);
            }
        }
    } else if constexpr (!EVEN) {
        MOE_LOAD_EXTRA();
    }
    if constexpr (!EVEN) {
        if (extra) {
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                acc[0][t] = mfma16(xw[0], xb[t], acc[0][t]);
                acc[1][t] = mfma16(xw[1], xb[t], acc[1][t]);
            }
        }
    }
#undef MOE_LOAD_EXTRA
#undef MOE_STEP_INDEX
#undef MOE_LOAD_A
#undef MOE_LOAD_B
#undef MOE_STAGE_B
#undef MOE_MMA_STEP
    __syncthreads();                                             // the staging tiles are reused for the reduction
    put_partials<2, NT, TT>(lds, acc, wave, lane);
}

// Stage 2 of one item.  Stage 1 leaves the block's rows of `act` as MFMA B-operand images, so a
// token fragment is one coalesced 1 KiB load straight into registers, like a weight fragment, with
// no LDS on the way.  A step is U K-steps (U = 2, 4 KiB of contiguous weights, when the number of
// K-steps is even and the token tiles leave room in the registers); the steps go round-robin over
// the wavefronts, 4 / U or 3 of them in flight for both operands, the weights issued before the
// wait for the block (they do not depend on stage 1).
// NW = 2: the item is a pair of adjacent tiles (64 output channels; their weights lie w_tile bytes apart) multiplied with the same token fragments: half as many items and `act`
// loads per block, twice the weight bytes in flight per workgroup.  Blocks of up to 16 rows (32
// in the 64-row launch) have the registers for it.  n_readers: calls of this function per block.
// Leaves the partial sums in LDS (put_partials); false: the wait for the block ran out and nothing was computed.
template <int NT, int TT, int U, bool STREAM, int NW>
__device__ __forceinline__ bool stream_item_down(const StreamArgs &a, const StageArgs &g, char *lds, int *s_ok,
                                                 const char *w, size_t w_tile, int item, int tile, int n_readers,
                                                 int wave, int lane) {
    asm volatile("" : "+v"(lane));                             // see wide_item
    constexpr int D = U == 2 ? 2 : NT > 2 ? 3 : 4;               // steps in flight that fit the registers
    constexpr int F = 2 * NW;                                    // weight fragments per K-step
    const uint32_t aoff = lane * 16;
    const char *bbase = reinterpret_cast<const char *>(g.B) + static_cast<size_t>(item) * a.act_block_bytes + aoff;
    const int n = (g.KS / U - wave + kWaves - 1) / kWaves;      // steps wave, wave+4, ... of this wavefront
    f32x4 acc[F][NT];
#pragma unroll
    for (int h = 0; h < F; ++h)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[h][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    bf16x8 wr[D][U][F], br[D][U][NT];
    const int last = n > 0 ? n - 1 : 0;
    const int rot = n > 0 ? static_cast<int>(static_cast<unsigned>(tile) % static_cast<unsigned>(n)) : 0;
#define MOE_STEP_INDEX(step)                                                                     \
        const int q_ = (step);                                                                   \
        int r_ = (q_ < last ? q_ : last) + rot;                                                  \
        r_ = r_ >= n ? r_ - n : r_;                                                              \
        const int s_ = wave + kWaves * r_;
#define MOE_LOAD_W(d, step)                                                                      \
    do {                                                                                         \
        MOE_STEP_INDEX(step)                                                                     \
        const char *ws_ = w + static_cast<size_t>(s_) * (U * 2048) + aoff;                       \
        _Pragma("unroll") for (int nw = 0; nw < NW; ++nw)                                        \
            _Pragma("unroll") for (int u = 0; u < U; ++u) {                                      \
                wr[d][u][2 * nw] = load_weights<STREAM>(ws_ + nw * w_tile + u * 2048);          \
                wr[d][u][2 * nw + 1] = load_weights<STREAM>(ws_ + nw * w_tile + u * 2048 + 1024); \
            }                                                                                    \
        asm volatile("" ::: "memory");                                                           \
    } while (0)
#define MOE_LOAD_T(d, step)                                                                      \
    do {                                                                                         \
        MOE_STEP_INDEX(step)                                                                     \
        const char *bs_ = bbase + static_cast<size_t>(s_) * (U * TT * 1024);                     \
        _Pragma("unroll") for (int u = 0; u < U; ++u)                                            \
            _Pragma("unroll") for (int t = 0; t < NT; ++t)                                       \
                br[d][u][t] = *reinterpret_cast<const bf16x8 *>(bs_ + (u * TT + t) * 1024);      \
        asm volatile("" ::: "memory");                                                           \
    } while (0)
#define MOE_MMA_STEP(d)                                                                          \
    do {                                                                                         \
        _Pragma("unroll") for (int u = 0; u < U; ++u)                                            \
            _Pragma("unroll") for (int t = 0; t < NT; ++t)                                       \
                _Pragma("unroll") for (int f = 0; f < F; ++f)                                    \
                    acc[f][t] = mfma16(wr[d][u][f], br[d][u][t], acc[f][t]);                     \
    } while (0)
#pragma unroll
    for (int d = 0; d < D; ++d)
        if (d < n) MOE_LOAD_W(d, d);
    if (!wait_block_ready(a, s_ok, item, tile, n_readers)) return false;
    if (n > 0) {
#pragma unroll
        for (int d = 0; d < D; ++d)
            if (d < n) MOE_LOAD_T(d, d);
        int i = 0;
        for (; i + 2 * D <= n; i += D) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                MOE_MMA_STEP(d);
                MOE_LOAD_W(d, i + d + D);
                MOE_LOAD_T(d, i + d + D);
            }
        }
        const int rem = n - i;                                   // 1 .. 2*D-1 steps left
#pragma unroll
        for (int d = 0; d < D; ++d) {
            if (d < rem) MOE_MMA_STEP(d);
            if (d < D - 1 && d + D < rem) { MOE_LOAD_W(d, i + d + D); MOE_LOAD_T(d, i + d + D); }
        }
#pragma unroll
        for (int d = 0; d < D - 1; ++d)
            if (D + d < rem) MOE_MMA_STEP(d);
    }
#undef MOE_STEP_INDEX
#undef MOE_LOAD_W
#undef MOE_LOAD_T
#undef MOE_MMA_STEP
    put_partials<F, NT, TT>(lds, acc, wave, lane);
    return true;
}

// ---------------------------------------------------------------------------------------------
// Slots with more requests than one block holds ("wide" slots): blocks of up to RT*16 rows as tiled
// GEMMs inside the same launch.  The streaming items above re-read a tile's weights for every block
// of rows and every item gathers its token rows again; here a workgroup computes RT*16 rows x 4
// packed weight tiles (64 channels of SiLU(gate)*up in stage 1, 128 output channels in stage 2),
// so the weights are fetched once per RT*16 rows and the token rows once per 4 tiles.
//
// Each of the 4 wavefronts owns one packed tile (two MFMA A fragments per K-step, read straight from
// global memory: the packed layout is the register image) and all rows: RT row tiles x 2
// accumulators.  Gate and up of a channel live in the same lane, so stage 1 needs no exchange between
// wavefronts, and a wavefront runs the whole K dimension (no split-K, no reduction).  The token rows
// (the B operand, shared by the 4 wavefronts) go through LDS: per K-tile of 64 columns the workgroup
// reads one 128-byte line of each row with whole-line loads (8 rows per instruction) into a
// double-buffered, XOR-swizzled tile, from which every wavefront reads the MFMA layout.  One
// barrier per K-tile; two K-tiles of both operands are in flight in registers.
//
// A wide block is led by the list entry whose first row is a multiple of RT*16 rows into the slot;
// the block's workgroups are the first ceil(tiles/4) ids of that entry (the others, and all ids of
// the slot's other entries, leave).  The intermediate of a wide block lives in the `act` region of
// its leading entry as [K-tile of stage 2 = 64 channels][row][128 bytes]: every 128-byte line has one
// writing workgroup, and stage 2 reads a K-tile of all rows as one contiguous run.  The hand-off is
// the one of the streaming items: counter and flags of the leading entry.
template <bool STAGE1, int RT, bool AHEAD>
__device__ __forceinline__ void wide_item(const StreamArgs &a, const StageArgs &g, char *lds, int *s_ok,
                                          int item, int group, int n_groups, int slot, int row0, int m, bool drain) {
    constexpr int kRing = 2;                                         // K-tiles of both operands in flight
    constexpr bool STREAM = false;                                   // a wide slot has several blocks: they share the tiles through L2
    constexpr int kPieces = RT * 16 * 8;                             // 16-byte pieces of one K-tile of the token tile
    constexpr int kLoadsB = (kPieces + kThreads - 1) / kThreads;
    constexpr int kBufBytes = RT * 16 * 128;
    // an opaque copy of the thread id: nothing derived from it is shared with (and hoisted above) the
    // other kinds of items, whose paths would then carry it in registers
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int wave = __builtin_amdgcn_readfirstlane(tid / MOE_WAVE), lane = tid % MOE_WAVE;
    int pt = group * kWaves + wave;
    const bool pt_ok = pt < g.tiles;
    pt = pt_ok ? pt : g.tiles - 1;
    const char *w = g.Wp + (static_cast<size_t>(slot) * g.tiles + pt) * g.KS * 2048 + lane * 16;
    const int rows_pad = (m + 15) & ~15;
    char *act_blk = reinterpret_cast<char *>(a.act) + static_cast<size_t>(item) * a.act_block_bytes;

    if constexpr (!STAGE1) {
        if (!wait_block_ready(a, s_ok, item, group, n_groups)) {
            const float qnan = __uint_as_float(0x7fc00000u);
            const f32x4 v = {qnan, qnan, qnan, qnan};
            const int c0 = group * 128, nc = (g.tiles * 32 - c0 < 128 ? g.tiles * 32 - c0 : 128) / 4;
            for (int i = tid; i < m * nc; i += kThreads)
                *reinterpret_cast<f32x4 *>(a.Yp + static_cast<size_t>(row0 + i / nc) * g.out_stride + c0 + (i % nc) * 4) = v;
            return;
        }
    }

    // token rows this thread fetches: piece q*256 + tid = row (q*32 + tid/8), 16-byte chunk tid%8 of the line
    const bool loader = kPieces >= kThreads || tid < kPieces;
    int req[kLoadsB];
#pragma unroll
    for (int q = 0; q < kLoadsB; ++q) {
        int r = q * (kThreads / 8) + (tid >> 3);
        r = r < m ? r : m - 1;
        req[q] = STAGE1 ? a.perm[row0 + r] : r;
    }
    asm volatile("" ::: "memory");
    const char *bp[kLoadsB];
    const size_t kt_stride = STAGE1 ? 128 : static_cast<size_t>(rows_pad) * 128;   // bytes a K-tile advances a row
    // LDS: row R at R*128, its 16-byte chunk c at ((c ^ ((R >> 1) & 7)) * 16): the 16 rows that one
    // fragment read touches then fall into 16 different bank groups (rows R and R+8 share R & 7)
    const uint32_t wr_lds = (tid >> 3) * 128 + (((tid & 7) ^ ((tid >> 4) & 7)) * 16);
    const uint32_t rd_row = (lane & 15) * 128, rd_sw = (lane >> 1) & 7, rd_g = lane >> 4;

    const int NKT = (g.KS + 1) >> 1;                                 // K-tiles of two K-steps (the last may hold one); >= 1
    f32x4 acc[RT][2];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) { acc[rt][0] = f32x4{0.f, 0.f, 0.f, 0.f}; acc[rt][1] = acc[rt][0]; }
    // K-tile i uses register set i % kRing and LDS buffer i % 2; loads past the last K-tile fetch the
    // last one again, so the steady-state loop has no branch around a load and the compiler counts
    // outstanding loads exactly.
    bf16x8 breg[kRing][kLoadsB];
    bf16x8 areg[kRing][2][2];                                        // [set][K-step of the tile][fragment]
    const int last = NKT - 1;

    // K-tile j: columns 64*j .. 64*j+63.  With an odd number of K-steps the last tile has only its
    // first half: its second K-step repeats the first (never multiplied) and chunks 4..7 of the
    // line, which lie past the row (stage 1) or were never written (stage 2), repeat chunks 0..3.
#define MOE_WIDE_LOAD_A(set, j)                                                                  \
    do {                                                                                         \
        const int j_ = (j) < last ? (j) : last;                                                  \
        const int s0_ = 2 * j_, s1_ = 2 * j_ + 1 < g.KS ? 2 * j_ + 1 : 2 * j_;                   \
        areg[set][0][0] = load_weights<STREAM>(w + static_cast<size_t>(s0_) * 2048);            \
        areg[set][0][1] = load_weights<STREAM>(w + static_cast<size_t>(s0_) * 2048 + 1024);     \
        areg[set][1][0] = load_weights<STREAM>(w + static_cast<size_t>(s1_) * 2048);            \
        areg[set][1][1] = load_weights<STREAM>(w + static_cast<size_t>(s1_) * 2048 + 1024);     \
        asm volatile("" ::: "memory");                                                           \
    } while (0)
#define MOE_WIDE_LOAD_B(set, j)                                                                  \
    do {                                                                                         \
        const int j_ = (j) < last ? (j) : last;                                                  \
        const size_t off_ = static_cast<size_t>(j_) * kt_stride - ((2 * j_ + 1 >= g.KS && (tid & 7) >= 4) ? 64 : 0); \
        if (loader) {                                                                            \
            _Pragma("unroll") for (int q = 0; q < kLoadsB; ++q)                                  \
                breg[set][q] = *reinterpret_cast<const bf16x8 *>(bp[q] + off_);                  \
        }                                                                                        \
        asm volatile("" ::: "memory");                                                           \
    } while (0)
#define MOE_WIDE_STAGE(set)                                                                      \
    do {                                                                                         \
        if (loader) {                                                                            \
            _Pragma("unroll") for (int q = 0; q < kLoadsB; ++q)                                  \
                *reinterpret_cast<bf16x8 *>(lds + ((set) & 1) * kBufBytes + q * (kThreads * 16) + wr_lds) = breg[set][q]; \
        }                                                                                        \
        asm volatile("" ::: "memory");                                                           \
    } while (0)
    // A K-tile's products.  AHEAD: the second K-step's fragments are read between the first one's products, one behind each row tile's,
    // instead of ahead of its own, where every wavefront waits for LDS a second time.  This launch alone, us: 32 blocks and no streams 82.8 ->
    // 81.6 (d_h = 2048, d_e = 1408, T = 1000) and 55.1 -> 54.0 (d_e = 768, T = 1500); 58 blocks beside streams (d_e = 1408, T = 1500) 105.6 ->
    // 103.5 with runs of one side 1.4 apart; up to 26 blocks beside streams (T = 500 to 1000, also d_h = 4096 and 7168) level, 0.99 to 1.00.
#define MOE_WIDE_READ(set, ss, r)                                                                \
    b_[r] = *reinterpret_cast<const bf16x8 *>(lds + ((set) & 1) * kBufBytes + (r) * 2048 + rd_row + (((4 * (ss) + rd_g) ^ rd_sw) * 16))
#define MOE_WIDE_MMA(set, full)                                                                  \
    do {                                                                                         \
        bf16x8 b_[RT];                                                                           \
        _Pragma("unroll") for (int r = 0; r < RT; ++r) MOE_WIDE_READ(set, 0, r);                 \
        if constexpr (AHEAD) { asm volatile("" ::: "memory"); __builtin_amdgcn_sched_barrier(0); } \
        _Pragma("unroll") for (int r = 0; r < RT; ++r) {                                         \
            acc[r][0] = mfma16(areg[set][0][0], b_[r], acc[r][0]);                               \
            acc[r][1] = mfma16(areg[set][0][1], b_[r], acc[r][1]);                               \
            if constexpr (AHEAD) {                                                               \
                if (full) MOE_WIDE_READ(set, 1, r);                                              \
                asm volatile("" ::: "memory");                                                   \
                __builtin_amdgcn_sched_barrier(0);                                               \
            }                                                                                    \
        }                                                                                        \
        if (full) {                                                                              \
            if constexpr (!AHEAD) {                                                              \
                _Pragma("unroll") for (int r = 0; r < RT; ++r) MOE_WIDE_READ(set, 1, r);         \
            }                                                                                    \
            _Pragma("unroll") for (int r = 0; r < RT; ++r) {                                     \
                acc[r][0] = mfma16(areg[set][1][0], b_[r], acc[r][0]);                           \
                acc[r][1] = mfma16(areg[set][1][1], b_[r], acc[r][1]);                           \
            }                                                                                    \
        }                                                                                        \
    } while (0)
    // The LDS buffer written here was last read in the multiply of K-tile i-2, which every wavefront
    // finished before the barrier of K-tile i-1.  full: both K-steps of the tile exist (a literal).
#define MOE_WIDE_STEP(set, i, full)                                                              \
    do {                                                                                         \
        MOE_WIDE_STAGE(set);                                                                     \
        MOE_WIDE_LOAD_B(set, (i) + kRing);                                                       \
        lds_barrier();                                                                           \
        MOE_WIDE_MMA(set, full);                                                                 \
        asm volatile("" ::: "memory");                                                           \
        MOE_WIDE_LOAD_A(set, (i) + kRing);                                                       \
    } while (0)

    const int n_full = g.KS >> 1;                                    // K-tiles with both K-steps
    int i = 0;
    // the weights do not wait for the requests' tokens to be known
    MOE_WIDE_LOAD_A(0, 0);
    MOE_WIDE_LOAD_A(1, 1);
#pragma unroll
    for (int q = 0; q < kLoadsB; ++q) {
        if constexpr (STAGE1)
            bp[q] = reinterpret_cast<const char *>(g.B) +
                    static_cast<size_t>(a.k_div(req[q])) * static_cast<uint32_t>(g.b_stride) * 2 + (tid & 7) * 16;
        else
            bp[q] = act_blk + static_cast<size_t>(req[q]) * 128 + (tid & 7) * 16;
    }
    MOE_WIDE_LOAD_B(0, 0);
    MOE_WIDE_LOAD_B(1, 1);
    // The first token rows are waited for here: inside the loop the compiler would leave as few loads in flight in every round as
    // there are behind these rows now (the weights of both K-tiles are in front of them, in the loop one K-tile's are).
    // drain: just that is wanted (kWideDrainWorkgroups).
    wait_loads<kLoadsB>();
    for (; i + 2 <= n_full; i += 2) {
        if (drain) wait_loads<kLoadsB>();
        MOE_WIDE_STEP(0, i, true);
        MOE_WIDE_STEP(1, i + 1, true);
    }
    const int rem = n_full - i;                                      // 0 .. 1
    if (rem > 0) MOE_WIDE_STEP(0, i, true);
    if (g.KS & 1) {
        if (rem == 0) MOE_WIDE_STEP(0, n_full, false);
        else MOE_WIDE_STEP(1, n_full, false);
    }
#undef MOE_WIDE_LOAD_A
#undef MOE_WIDE_LOAD_B
#undef MOE_WIDE_STAGE
#undef MOE_WIDE_READ
#undef MOE_WIDE_MMA
#undef MOE_WIDE_STEP

    // lane l holds, per row tile, 4 consecutive channels (l/16)*4.. of row (l%16) of the tile
    if (pt_ok) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            const int r = rt * 16 + (lane & 15);
            if (r >= m) continue;
            if constexpr (STAGE1) {
                const f32x4 gt = acc[rt][0], up = acc[rt][1];
                const uint64_t o = moe::f32x2_to_bf16x2(silu_mul(gt[0], up[0]), silu_mul(gt[1], up[1])) |
                                   static_cast<uint64_t>(moe::f32x2_to_bf16x2(silu_mul(gt[2], up[2]), silu_mul(gt[3], up[3]))) << 32;
                uint64_t *dst = reinterpret_cast<uint64_t *>(act_blk + (static_cast<size_t>(group) * rows_pad + r) * 128 +
                                                             wave * 32 + (lane >> 4) * 8);
                __hip_atomic_store(dst, o, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            } else {
                float *dst = a.Yp + static_cast<size_t>(row0 + r) * g.out_stride + pt * 32 + (lane >> 4) * 4;
                *reinterpret_cast<f32x4 *>(dst) = acc[rt][0];
                *reinterpret_cast<f32x4 *>(dst + 16) = acc[rt][1];
            }
        }
    }
    if constexpr (STAGE1) announce_tiles(a, item, n_groups);
}

// The same in the launch of large batches (ffn_big_kernel: two workgroups a CU): blocks of up to 64 or 128 rows, two packed tiles a
// wavefront, eight a workgroup.  A token fragment read from LDS then serves four matrix instructions, and a K-tile's operands
// serve twice as many: matrix cores : L1 : LDS = 512 : 640 : 320 cycles a K-tile with 64 rows and 1024 : 768 : 640 with 128, where
// one packed tile a wavefront and 64 rows need 256 : 384 : 320 and such workgroups mostly add the three up.  Weights: a ring of four
// (128 rows: two) K-tiles in registers, each K-step's part requested again as soon as it is multiplied.  Token rows: two (one)
// K-tiles ahead in registers, a double buffer in LDS that is written between the two K-steps of the K-tile before; one barrier a K-tile.
template <bool STAGE1, int RT>
__device__ __forceinline__ void wide_item2(const StreamArgs &a, const StageArgs &g, char *lds, int *s_ok,
                                           int item, int group, int n_groups, int slot, int row0, int m) {
    constexpr int P = 2;                                             // packed tiles of a wavefront
    constexpr int F = 2 * P;                                         // weight fragments of a K-step
    constexpr int kLoadsB = RT * 16 * 8 / kThreads;                  // 16-byte pieces of a K-tile of the token rows per thread
    constexpr int kBufBytes = RT * 16 * 128;
    constexpr int kRing = RT == 4 ? 4 : 2;                           // K-tiles of weights in flight
    constexpr int kRingB = RT == 4 ? 2 : 1;                      // K-tiles of token rows in flight
    static_assert(RT % 4 == 0, "whole loads per thread, row tiles in groups of four");
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));                                    // see wide_item
    const int wave = __builtin_amdgcn_readfirstlane(tid / MOE_WAVE), lane = tid % MOE_WAVE;
    const int pt0 = (group * kWaves + wave) * P;
    const char *w[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int pt = pt0 + p < g.tiles ? pt0 + p : g.tiles - 1;
        w[p] = g.Wp + (static_cast<size_t>(slot) * g.tiles + pt) * g.KS * 2048;
    }
    const uint32_t aoff = lane * 16;
    const int rows_pad = (m + 15) & ~15;
    char *act_blk = reinterpret_cast<char *>(a.act) + static_cast<size_t>(item) * a.act_block_bytes;

    if constexpr (!STAGE1) {
        if (!wait_block_ready(a, s_ok, item, group, n_groups)) {
            const float qnan = __uint_as_float(0x7fc00000u);
            const f32x4 v = {qnan, qnan, qnan, qnan};
            const int cols = kWaves * P * 32, c0 = group * cols, nc = (g.tiles * 32 - c0 < cols ? g.tiles * 32 - c0 : cols) / 4;
            for (int i = tid; i < m * nc; i += kThreads)
                *reinterpret_cast<f32x4 *>(a.Yp + static_cast<size_t>(row0 + i / nc) * g.out_stride + c0 + (i % nc) * 4) = v;
            return;
        }
    }
    // token rows this thread fetches: piece q*256 + tid = row (q*32 + tid/8), 16-byte chunk tid%8 of the line
    uint32_t boff[kLoadsB];
#pragma unroll
    for (int q = 0; q < kLoadsB; ++q) {
        int r = q * (kThreads / 8) + (tid >> 3);
        r = r < m ? r : m - 1;
        boff[q] = STAGE1 ? static_cast<uint32_t>(a.perm[row0 + r]) : static_cast<uint32_t>(r) * 128 + (tid & 7) * 16;
    }
    asm volatile("" ::: "memory");
    const char *bbase = STAGE1 ? reinterpret_cast<const char *>(g.B) : act_blk;
    const size_t kt_stride = STAGE1 ? 128 : static_cast<size_t>(rows_pad) * 128;   // bytes a K-tile advances a row
    // LDS as in wide_item
    const uint32_t wr_lds = (tid >> 3) * 128 + (((tid & 7) ^ ((tid >> 4) & 7)) * 16);
    const uint32_t rd_row = (lane & 15) * 128, rd_sw = (lane >> 1) & 7, rd_g = lane >> 4;
    const uint32_t half_back = (tid & 7) >= 4 ? 64 : 0;              // see MOE_W2_LOAD_B

    const int NKT = (g.KS + 1) >> 1;                                 // K-tiles of two K-steps (the last may hold one); >= 1
    const int last = NKT - 1;
    f32x4 acc[RT][F];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int f = 0; f < F; ++f) acc[rt][f] = f32x4{0.f, 0.f, 0.f, 0.f};
    bf16x8 areg[kRing][2][F];                                        // [K-tile % kRing][K-step][fragment]
    bf16x8 breg[kRingB][kLoadsB];
    // Loads past the last K-tile fetch the last one again; the second K-step of a last half K-tile repeats the first.
#define MOE_W2_LOAD_A(set, ss, j)                                                                \
    do {                                                                                         \
        const int j_ = (j) < last ? (j) : last;                                                  \
        const int s_ = 2 * j_ + (ss) < g.KS ? 2 * j_ + (ss) : 2 * j_;                            \
        _Pragma("unroll") for (int p = 0; p < P; ++p) {                                          \
            const char *ws_ = w[p] + static_cast<size_t>(s_) * 2048;                             \
            areg[set][ss][2 * p] = load_weights<false>(ws_ + aoff);                              \
            areg[set][ss][2 * p + 1] = load_weights<false>(ws_ + 1024 + aoff);                   \
        }                                                                                        \
        asm volatile("" ::: "memory");                                                           \
    } while (0)
    // chunks 4..7 of the line of a half K-tile, which lie past the row or were never written, repeat chunks 0..3
#define MOE_W2_LOAD_B(d, j)                                                                       \
    do {                                                                                         \
        const int j_ = (j) < last ? (j) : last;                                                  \
        const char *bs_ = bbase + static_cast<size_t>(j_) * kt_stride;                           \
        const uint32_t back_ = 2 * j_ + 1 >= g.KS ? half_back : 0;                               \
        _Pragma("unroll") for (int q = 0; q < kLoadsB; ++q)                                      \
            breg[(d) % kRingB][q] = *reinterpret_cast<const bf16x8 *>(bs_ + (boff[q] - back_));  \
        asm volatile("" ::: "memory");                                                           \
    } while (0)
#define MOE_W2_STAGE(buf, d)                                                                        \
    do {                                                                                         \
        _Pragma("unroll") for (int q = 0; q < kLoadsB; ++q)                                      \
            *reinterpret_cast<bf16x8 *>(lds + (buf) * kBufBytes + q * (kThreads * 16) + wr_lds) = breg[(d) % kRingB][q]; \
        asm volatile("" ::: "memory");                                                           \
    } while (0)
#define MOE_W2_MMA(set, ss)                                                                      \
    do {                                                                                         \
        _Pragma("unroll") for (int r0_ = 0; r0_ < RT; r0_ += 4) {                                \
            bf16x8 b_[4];                                                                        \
            _Pragma("unroll") for (int r4 = 0; r4 < 4; ++r4)                                     \
                b_[r4] = *reinterpret_cast<const bf16x8 *>(                                      \
                    lds + ((set) & 1) * kBufBytes + (r0_ + r4) * 2048 + rd_row + (((4 * (ss) + rd_g) ^ rd_sw) * 16)); \
            _Pragma("unroll") for (int r4 = 0; r4 < 4; ++r4)                                     \
                _Pragma("unroll") for (int f = 0; f < F; ++f)                                    \
                    acc[r0_ + r4][f] = mfma16(areg[set][ss][f], b_[r4], acc[r0_ + r4][f]);       \
        }                                                                                        \
        asm volatile("" ::: "memory");                                                           \
    } while (0)
    // The buffer written here was last read in K-tile i-1, which every wavefront finished before the barrier at its end.
    // set = i % kRing, a literal.
#define MOE_W2_STEP(set, i)                                                                      \
    do {                                                                                         \
        MOE_W2_MMA(set, 0);                                                                      \
        MOE_W2_LOAD_A(set, 0, (i) + kRing);                                                      \
        MOE_W2_STAGE(1 - ((set) & 1), (set) + 1);                                                \
        MOE_W2_LOAD_B((set) + 1, (i) + 1 + kRingB);                                              \
        MOE_W2_MMA(set, 1);                                                                      \
        MOE_W2_LOAD_A(set, 1, (i) + kRing);                                                      \
        lds_barrier();                                                                           \
    } while (0)

    MOE_W2_LOAD_A(0, 0, 0);
    MOE_W2_LOAD_A(0, 1, 0);
    if constexpr (STAGE1) {
#pragma unroll
        for (int q = 0; q < kLoadsB; ++q)
            boff[q] = a.k_div(boff[q]) * static_cast<uint32_t>(g.b_stride) * 2 + (tid & 7) * 16;
    }
    MOE_W2_LOAD_B(0, 0);
#pragma unroll
    for (int d = 1; d < kRing; ++d) {
        MOE_W2_LOAD_A(d, 0, d);
        MOE_W2_LOAD_A(d, 1, d);
        if (d < kRingB) MOE_W2_LOAD_B(d, d);
    }
    MOE_W2_STAGE(0, 0);
    MOE_W2_LOAD_B(0, kRingB);
    lds_barrier();
    // the last K-tiles: their weights have been requested, the last one may be half
#define MOE_W2_TAIL(set, i)                                                                      \
    do {                                                                                         \
        MOE_W2_MMA(set, 0);                                                                      \
        if ((i) < last) {                                                                        \
            MOE_W2_STAGE(1 - ((set) & 1), (set) + 1);                                            \
            if (kRing > kRingB + 1) MOE_W2_LOAD_B((set) + 1, (i) + 1 + kRingB);                  \
        }                                                                                        \
        if (2 * (i) + 1 < g.KS) MOE_W2_MMA(set, 1);                                              \
        lds_barrier();                                                                           \
    } while (0)
    const int n_full = g.KS >> 1;                                    // K-tiles with both K-steps
    int i = 0;
    for (; i + kRing <= n_full; i += kRing) {
        MOE_W2_STEP(0, i);
        MOE_W2_STEP(1, i + 1);
        if constexpr (kRing == 4) {
            MOE_W2_STEP(2, i + 2);
            MOE_W2_STEP(3, i + 3);
        }
    }
    // at most kRing K-tiles are left, wave-uniform
    if (i <= last) MOE_W2_TAIL(0, i);
    if (i + 1 <= last) MOE_W2_TAIL(1, i + 1);
    if constexpr (kRing == 4) {
        if (i + 2 <= last) MOE_W2_TAIL(2, i + 2);
        if (i + 3 <= last) MOE_W2_TAIL(3, i + 3);
    }
#undef MOE_W2_TAIL
#undef MOE_W2_LOAD_A
#undef MOE_W2_LOAD_B
#undef MOE_W2_STAGE
#undef MOE_W2_MMA
#undef MOE_W2_STEP

    // lane l holds, per row tile, 4 consecutive channels (l/16)*4.. of row (l%16) of each fragment
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        const int r = rt * 16 + (lane & 15);
        if (r >= m) continue;
#pragma unroll
        for (int p = 0; p < P; ++p) {
            if (pt0 + p >= g.tiles) continue;
            if constexpr (STAGE1) {
                const f32x4 gt = acc[rt][2 * p], up = acc[rt][2 * p + 1];
                const uint64_t o = moe::f32x2_to_bf16x2(silu_mul(gt[0], up[0]), silu_mul(gt[1], up[1])) |
                                   static_cast<uint64_t>(moe::f32x2_to_bf16x2(silu_mul(gt[2], up[2]), silu_mul(gt[3], up[3]))) << 32;
                // [K-tile of stage 2 = 4 packed tiles][row][128 bytes]
                uint64_t *dst = reinterpret_cast<uint64_t *>(act_blk + (static_cast<size_t>((pt0 + p) >> 2) * rows_pad + r) * 128 +
                                                             ((pt0 + p) & 3) * 32 + (lane >> 4) * 8);
                __hip_atomic_store(dst, o, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            } else {
                float *dst = a.Yp + static_cast<size_t>(row0 + r) * g.out_stride + (pt0 + p) * 32 + (lane >> 4) * 4;
                *reinterpret_cast<f32x4 *>(dst) = acc[rt][2 * p];
                *reinterpret_cast<f32x4 *>(dst + 16) = acc[rt][2 * p + 1];
            }
        }
    }
    if constexpr (STAGE1) announce_tiles(a, item, n_groups);
}

// A slot with more than kWideMin requests is wide.  Its rows are cut into blocks of WR = 64 rows (a block
// of 128 rows needs 64 accumulator registers more than the streaming items leave at three workgroups
// per CU; large batches take ffn_big_kernel instead).
constexpr int kWideMin = 64;
// A wavefront of a wide workgroup runs its tile's whole K dimension, one round trip per K-tile (about
// kWideTileNs each), so a wide workgroup lasts much longer than a streaming item.  Wide blocks pay off
//  - when a batch has enough of them to fill the chip with such workgroups: (64-row blocks of the wide
//    slots, from the list's header) x (first-stage workgroups per block) >= kWideMinWorkgroups; or
//  - from kWideMinHidden workgroups on, when the rest of the launch lasts long enough to hide them (they
//    come first in the list and start with the launch): the time the launch needs to stream one expert
//    per list entry at kStreamBytesPerNs must exceed 5/4 of the K-tiles of both stages x kWideTileNs.
// Otherwise the wide slots are cut into streaming items like the others.  Every workgroup takes the
// decision from the same numbers.  A caller's threshold replaces the first rule and switches the
// second off.
constexpr int kWideMinWorkgroups = 256;
constexpr int kWideMinHidden = 64;
constexpr long long kWideTileNs = 900, kStreamBytesPerNs = 7000;
// beside_ns: the same for the other expert set of a launch that runs two.
__device__ __forceinline__ long long stream_ns(int blocks, int ks1, int ks2) {
    // an expert's three matrices: 3 * d_h * d_e bf16 = ks1 * ks2 * 32 * 32 * 6 bytes
    return static_cast<long long>(blocks) * ks1 * ks2 * (32 * 32 * 6) / kStreamBytesPerNs;
}
__device__ __forceinline__ bool wide_on(int4 head, int groups1, int override_min, int ks1, int ks2, long long beside_ns = 0) {
    const int wgs = head.z * groups1;
    if (override_min > 0) return wgs >= override_min;
    if (wgs >= kWideMinWorkgroups) return true;
    if (wgs < kWideMinHidden) return false;
    const long long chain_ns = static_cast<long long>((ks1 + 1) / 2 + (ks2 + 1) / 2) * kWideTileNs;
    return 4 * (stream_ns(head.x, ks1, ks2) + beside_ns) >= 5 * chain_ns;
}
// Wide items let their ring of loads run empty every two K-tiles (drain) when there are more workgroups of their second stage than
// this; at most that many are a chain of round trips to memory each, which an empty ring lengthens (us, drained and not: 256 and 128
// workgroups of the two stages, d_h = d_e = 2048, 500 rows of one slot 34.7 and 29.4; 256 and 256, 4096 x 2048 48.7 and 40.2; 512 and
// 128, 2048 x 4096 52.7 and 47.5; 240 and 320, 4096 x 1536 60.6 and 57.5).  With more of them the blocks of a slot drift apart without
// it and fetch the expert's tiles one by one (768 and 768, 4096 x 2048 130 and 148; 384 and 1536, 8192 x 1024 160 and 171; 544 and
// 816, 3072 x 1024 88 and 90).  So they do where as many streaming blocks hide the wide ones and want the memory for themselves
// (d_h = 7168, d_e = 2048, T = 512 236 and 240).  Taken by the wide items alone: ahead of all items the rule costs those 1-3 %.
constexpr int kWideDrainWorkgroups = 352;
struct WideBlocks { int all, wide; };    // entries of the list (and of one beside it), 64-row blocks of the wide slots
// BR: rows of a list entry
template <int BR>
__device__ __forceinline__ bool wide_drains(WideBlocks n, int tiles2) {
    return n.wide * ((tiles2 + kWaves - 1) / kWaves) > kWideDrainWorkgroups || n.all - n.wide * (64 / BR) >= n.wide;
}
// The workgroups of a wide slot (ids in groups of ids8 * 8 per block: the block's, tile = 0 .. ids8 * 8 - 1) run the slot's nb blocks
// x groups of tiles; the others leave.
// Workgroup ids go round-robin over the eight XCDs, so tile % 8 is the XCD and (leader index, tile / 8)
// the place in that XCD's start order.  The XCDs take runs of the pairs (group, block), block-fastest, as even as they
// come and the longer ones first from XCD `turn` on (slots of few pairs would otherwise meet on the first XCDs: 20 slots of 150 rows,
// d_h = 4096, d_e = 1536, T = 700 303 -> 266 us): the blocks of one group of tiles start next to each other on one XCD, walk the expert's tiles side by side, and all but the first
// find them in that L2.  (Group-fastest, the natural order of the ids, put the sibling blocks tiles_pad / 8
// starts apart: on a busy chip that is longer than a line survives in a streaming L2, and every block of a
// slot fetched the expert from memory again.)  False: this workgroup has none.
struct WidePair { int group, block; };
__device__ __forceinline__ bool deal_wide(int leader, int tile, int ids8, int nb, int groups, int turn, WidePair &pair) {
    const int place = leader * ids8 + (tile >> 3);                   // in the XCD's start order, within the slot
    const int pairs = nb * groups, x = (tile - turn) & 7, each = pairs >> 3, more = pairs & 7;
    if (place >= each + (x < more ? 1 : 0)) return false;
    const int idx = x * each + (x < more ? x : more) + place;
    pair = {idx / nb, idx % nb};
    return true;
}

// In the launches of smaller batches: one entry leads each block of WR rows; all other workgroups of the slot's entries leave.
// BR = rows per list entry.
template <bool STAGE1, int WR, int BR>
__device__ __forceinline__ void run_wide(const StreamArgs &a, const StageArgs &g, char *lds, int *s_ok, int item,
                                         int tile, int4 ent, WideBlocks n) {
    const int slot = ent.x, hi = ent.z, lo = ent.w;
    if ((ent.y - lo) % WR != 0) return;                              // not the leading entry of a wide block
    const int groups = (g.tiles + kWaves - 1) / kWaves;              // workgroups of a block in this stage
    const int leader = (ent.y - lo) / WR;                            // which of the slot's blocks this entry leads
    WidePair pair;
    if (!deal_wide(leader, tile, g.tiles_pad >> 3, (hi - lo + WR - 1) / WR, groups, (item / (WR / BR) - leader) * groups, pair)) return;
    item += (pair.block - leader) * (WR / BR);                       // the block's leading entry: its control lines and `act`
    const int row0 = lo + pair.block * WR;
    const int m = hi - row0 < WR ? hi - row0 : WR;
    const int rt = (m + 15) >> 4;
    const bool drain = wide_drains<BR>(n, a.s[1].tiles);
    // up to 16 rows as two row tiles (one kind of item less; slots of 72 rows: 58 -> 61 us at d_h = 2048, d_e = 768, 173 -> 163 at
    // d_h = 4096, d_e = 1536)
    // The 32-row launch is without it: compiled for long lists it would spill 3 or 14 registers.  Its other instantiations would not; steps
    // there measured 0.98 to 1.00 with it (d_h = 2048, d_e = 1408, T = 256 63.1 -> 61.9 us; d_h = 7168 with a shared expert, T = 256
    // 226.9 -> 225.4; eleven others level).
    constexpr bool kAhead = BR == 64;
    if (rt <= 2) wide_item<STAGE1, 2, kAhead>(a, g, lds, s_ok, item, pair.group, groups, slot, row0, m, drain);
    else wide_item<STAGE1, 4, kAhead>(a, g, lds, s_ok, item, pair.group, groups, slot, row0, m, drain);
}

// EVEN: this stage has an even number of K-steps
// ent, the block's work list entry: {slot, first row, end of the slot's rows, first of the slot's rows}
template <bool STAGE1, bool EVEN, int TT>
__device__ __forceinline__ void run_stream_item(const StreamArgs &a, const StageArgs &g, char *lds, int *s_ok, int item, int tile,
                                                int4 ent) {
    if (tile >= g.items) return;                                 // ids that pad the tiles to a multiple of 8
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / MOE_WAVE), lane = threadIdx.x % MOE_WAVE;
    const int slot = ent.x, row0 = ent.y, hi = ent.z;
    // in the 64-row launch a stage-2 workgroup owns a pair of tiles (larger batches: the pairs halve
    // the workgroup turnover of the second stage; small batches want every tile on a workgroup of its own)
    constexpr bool kPairs = !STAGE1 && TT == 4;
    if constexpr (kPairs) tile *= 2;
    const char *w = g.Wp + (static_cast<size_t>(slot) * g.tiles + tile) * g.KS * 2048;
    const int m = hi - row0;
    const bool single = m <= TT * 16 && row0 == ent.w;                  // the slot's only block
    // Loads of a slot's only block carry the streaming hint, those of a slot with several do not (load_weights): its last,
    // partly filled block is computed with its row tiles rounded up to a power of two, to keep the instructions few.
    if constexpr (!STAGE1) {
        int nt = ((m < TT * 16 ? m : TT * 16) + 15) >> 4;                // 16-row token tiles that hold requests
        if (TT == 4 && !single) nt = nt <= 2 ? 2 : 4;
        constexpr int U = EVEN ? 2 : 1;
        const size_t tile_bytes = static_cast<size_t>(g.KS) * 2048;
        // 64-row launch: blocks of up to 32 rows multiply both tiles of the pair at once, larger ones one after the other
        // (every workgroup of a block takes the same branch, so the block's readers are counted the same way by all).
        // An odd number of tiles leaves the last one alone: its pair is itself and is not stored.
        const bool two = kPairs && tile + 1 < g.tiles;
        const bool paired = kPairs && nt <= 2;
        const int passes = kPairs && !paired && two ? 2 : 1, n_readers = paired ? g.items : g.tiles;
        for (int pass = 0; pass < passes; ++pass) {
            if (pass) __syncthreads();                                   // the LDS buffer is reused
            const int t = tile + pass;
            const char *w_ = w + pass * tile_bytes;
            bool ok;
#define MOE_DOWN(NT, U_, NW, STREAM) stream_item_down<NT, TT, U_, STREAM, NW>(a, g, lds, s_ok, w_, two ? tile_bytes : 0, item, t, n_readers, wave, lane)
            if constexpr (TT == 2) {
                if (single) ok = nt == 1 ? MOE_DOWN(1, U, 1, true) : MOE_DOWN(2, U, 1, true);
                else ok = nt == 1 ? MOE_DOWN(1, U, 1, false) : MOE_DOWN(2, U, 1, false);
            } else if (single) {
                if (nt == 1) ok = MOE_DOWN(1, U, 2, true);
                else if (nt == 2) ok = MOE_DOWN(2, U, 2, true);
                else if (nt == 3) ok = MOE_DOWN(3, 1, 1, true);
                else ok = MOE_DOWN(4, 1, 1, true);
            } else {
                ok = nt == 2 ? MOE_DOWN(2, U, 2, false) : MOE_DOWN(4, 1, 1, false);
            }
#undef MOE_DOWN
            const int nw = paired && two ? 2 : 1;                        // tiles to store
            if (ok) {
                __syncthreads();
                store_rows<TT>(a, g, lds, 2 * nw, nt, t, row0, hi);
            } else {
                for (int q = 0; q < nw; ++q) store_nan_rows(a, g, t + q, row0, m < TT * 16 ? m : TT * 16);
            }
        }
    } else {
        int halves = ((m < TT * 16 ? m : TT * 16) + 7) >> 3;             // 8-row halves that hold requests
        if (!single) halves = halves <= 2 ? 2 : halves <= 4 ? 4 : 8;
#define MOE_CASE(NH, STREAM) case NH: stream_item_lines<NH, TT, STREAM, EVEN>(a, g, lds, w, tile, row0, hi, wave, lane); break;
        if constexpr (TT == 2) {
            if (single) switch (halves) { MOE_CASE(1, true) MOE_CASE(2, true) MOE_CASE(3, true) MOE_CASE(4, true) }
            else switch (halves) { MOE_CASE(2, false) MOE_CASE(4, false) }
        } else {
            if (single) switch (halves) { MOE_CASE(1, true) MOE_CASE(2, true) MOE_CASE(3, true) MOE_CASE(4, true)
                                          MOE_CASE(5, true) MOE_CASE(6, true) MOE_CASE(7, true) MOE_CASE(8, true) }
            else switch (halves) { MOE_CASE(2, false) MOE_CASE(4, false) MOE_CASE(8, false) }
        }
#undef MOE_CASE
        __syncthreads();
        store_act<TT>(a, lds, (halves + 1) >> 1, item, tile, row0, hi);
    }
    if (STAGE1) announce_tiles(a, item, g.tiles);
}

// wide: slots with more than kWideMin requests are wide blocks (n of them); otherwise every slot is cut into streaming items.
template <bool STAGE1, bool EVEN, int TT, int WR>
__device__ __forceinline__ void run_item(const StreamArgs &a, const StageArgs &g, char *lds, int *s_ok, int wide,
                                         WideBlocks n, int item, int tile, int4 ent) {
    if (wide && ent.z - ent.w > kWideMin) run_wide<STAGE1, WR, TT * 16>(a, g, lds, s_ok, item, tile, ent, n);
    else run_stream_item<STAGE1, EVEN, TT>(a, g, lds, s_ok, item, tile, ent);
}

// 1-D grid sized for the worst case (at most kFfnLaneBlocks blocks).  With B = min(the batch's number of
// blocks, kFfnLaneBlocks), ids below B*tiles_pad(1) are the stage-1 workgroups (id = block * tiles_pad +
// tile), the next B*tiles_pad(2) ids the stage-2 workgroups, and the rest leave at once.  Workgroups are dispatched in id order, so a
// stage-2 workgroup is started after every stage-1 workgroup, and go to the XCDs round-robin, so
// the blocks of one tile of a slot (ids tiles_pad apart, a multiple of 8) run on the same XCD at
// about the same time: the tile's weights come from HBM once and are shared through that XCD's
// L2.  EVEN1 / EVEN2: a stage has an even number of K-steps.
// TT = token tiles per block (2: blocks of 32 rows, 4 workgroups per CU; 4: blocks of 64 rows, whose
// larger register set allows 3 per CU).  WRAP: the list can be longer than kFfnLaneBlocks.
template <bool EVEN1, bool EVEN2, int TT, int WR, bool WRAP>
__global__ __launch_bounds__(kThreads, TT == 2 ? 4 : 3)
void ffn_stream_kernel(StreamArgs a) {
    // split-K reduction buffer [4 waves][2][TT][64] x 16 B, which the whole-line path also uses as
    // its per-wavefront staging tiles during the K loop
    __shared__ __attribute__((aligned(16))) char lds[kWaves * 2 * TT * MOE_WAVE * 16];
    static_assert(kWaves * TT * 2048 <= sizeof(lds), "staging tiles must fit in the reduction buffer");
    static_assert(2 * WR * 128 <= sizeof(lds), "the two token tiles of a wide block must fit");
    __shared__ unsigned long long s_visit;                       // WRAP
    __shared__ int s_ok;
    {
        // ids are decoded with the number of blocks the batch really has, so that the surplus of
        // the worst-case grid comes after all the work of both stages
        // The header, the workspace's options and the entry this workgroup has if it is a stage-1 workgroup of a block with
        // workgroups of its own, all requested at once (an entry past the end of the list is never used).  One after the other,
        // with the weights behind the requests' tokens and divisions in between, they kept every workgroup from its first
        // operand for another 1.5 us: a layer step at d_h = 2048 with 17 blocks of up to 32 rows 37.1 -> 36.5 us, with odd numbers of
        // K-steps 59.1 -> 57.7.
        const unsigned item1 = a.s[0].pad_div(blockIdx.x);
        const int4 head = load_const(a.blocks, 0);
        const int4 ent1 = load_const(a.blocks, 1 + item1 < a.list_last ? 1 + item1 : a.list_last);
        const int wide_min = load_const(a.ctrl, 0).w;
        asm volatile("" ::"s"(head.x), "s"(ent1.x), "s"(ent1.y), "s"(ent1.z), "s"(ent1.w), "s"(wide_min));   // here, not behind the branches
        if (head.y != TT * 16) {
            // the list was cut for another block size (made for a different T): refuse, visibly
            if (threadIdx.x == 0 && blockIdx.x == 0)
                __hip_atomic_fetch_or(a.ctrl + moe::kCtrlStatus, 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return;
        }

        // Up to kFfnLaneBlocks blocks have workgroups of their own; a longer list wraps around (the
        // workgroup of block b also takes blocks b + kFfnLaneBlocks, ..., at most 64 of them), which
        // keeps the worst-case grid of large batches small.  A stage-1 workgroup never waits, and all of them are started
        // before any stage-2 workgroup, so every flag a stage-2 workgroup waits for is raised.
        // header word 3 of the workspace (wide_min): the caller's threshold for wide blocks (0 = default)
        const int wide = wide_on(head, (a.s[0].tiles + kWaves - 1) / kWaves, wide_min, a.s[0].KS, a.s[1].KS);
        const WideBlocks n = {head.x, head.z};
        const unsigned n_blocks = static_cast<unsigned>(head.x);
        const unsigned lanes = n_blocks < moe::kFfnLaneBlocks ? n_blocks : moe::kFfnLaneBlocks;
        const unsigned n1 = lanes * a.s[0].tiles_pad, n2 = lanes * a.s[1].tiles_pad;
        const auto own_item = [&] {
            if (blockIdx.x < n1) {
                run_item<true, EVEN1, TT, WR>(a, a.s[0], lds, &s_ok, wide, n, item1, blockIdx.x - item1 * a.s[0].tiles_pad, ent1);
            } else if (blockIdx.x - n1 < n2) {
                const unsigned id = blockIdx.x - n1, item = a.s[1].pad_div(id);
                run_item<false, EVEN2, TT, WR>(a, a.s[1], lds, &s_ok, wide, n, item, id - item * a.s[1].tiles_pad, load_const(a.blocks, 1 + item));
            }
        };
        if constexpr (!WRAP) {
            own_item();
        } else {
            if (n_blocks <= lanes) {
                own_item();              // as without WRAP: the loop's copy of the tiled-GEMM items is up to 4 % slower
                return;
            }
            if (blockIdx.x >= n1 + n2) return;
            const bool s1 = blockIdx.x < n1;
            const unsigned id0 = s1 ? blockIdx.x : blockIdx.x - n1;
            // a long list: the first wavefront looks at all the blocks of this workgroup at once (lane l:
            // block + l*lanes) and the workgroup then visits only those that are its own to compute
            const unsigned tp = s1 ? a.s[0].tiles_pad : a.s[1].tiles_pad, item0 = s1 ? item1 : a.s[1].pad_div(id0);
            // (ids that pad the tiles to a multiple of 8 stay: the wide slots use them)
            if (threadIdx.x < MOE_WAVE) {
                const unsigned b = item0 + threadIdx.x * lanes;
                // entries of wide slots that lead no block are not visited
                bool mine = false;
                if (b < n_blocks) {
                    const int4 e = reinterpret_cast<const int4 *>(a.blocks)[1 + b];
                    mine = !wide || e.z - e.w <= kWideMin || (e.y - e.w) % WR == 0;
                }
                const unsigned long long m = __ballot(mine);
                if (threadIdx.x == 0) s_visit = m;
            }
            __syncthreads();
            unsigned long long visit = static_cast<unsigned>(__builtin_amdgcn_readfirstlane(static_cast<int>(s_visit))) |
                                       static_cast<unsigned long long>(static_cast<unsigned>(
                                           __builtin_amdgcn_readfirstlane(static_cast<int>(s_visit >> 32)))) << 32;
            bool first = true;
#pragma unroll 1
            while (visit) {
                const unsigned l = static_cast<unsigned>(__builtin_ctzll(visit));
                visit &= visit - 1;
                if (!first) __syncthreads();                         // the LDS buffer is reused
                first = false;
                // opaque copies: what the items derive from these is not to be computed ahead of the loop for all kinds
                // of items at once (hundreds of spilled scalars)
                StageArgs g = s1 ? a.s[0] : a.s[1];
                asm volatile("" : "+s"(g.KS), "+s"(g.tiles), "+s"(g.tiles_pad), "+s"(g.items));
                const unsigned item = item0 + l * lanes;
                const int4 ent = load_const(a.blocks, 1 + item);
                if (s1) run_item<true, EVEN1, TT, WR>(a, g, lds, &s_ok, wide, n, item, id0 - item0 * tp, ent);
                else run_item<false, EVEN2, TT, WR>(a, g, lds, &s_ok, wide, n, item, id0 - item0 * tp, ent);
            }
        }
    }
}

// The routed experts (set 0) and a shared expert (set 1, one slot that every token visits: k = 1) in one launch.  On its own
// the shared expert's few hundred rows are a chain of K-tiles that neither the memory nor the matrix cores limit; here it
// runs beside the routed experts' stream, which leaves both idle (T = 256, d_h = 7168, d_e = 2048, shared width 2048: the
// two launches 168 + 77 us).  Its first-stage workgroups have the lowest ids, because their chains are the longest, and
// the numbers of its blocks and of those ids follow from T; then the routed first stage, and the second stages in
// the same order, so that again no workgroup waits for one with a higher id.  Every block has workgroups of its own, and
// the second stages have the same parity of K-steps.  Layer steps with a shared expert, two FFN launches and one, us, means of three
// inputs: T = 256 as above 282 -> 234, T = 8 109 -> 95; d_h = 2048, d_e = 1408, shared width 1408: T = 8 43 -> 34, T = 128 63 -> 56,
// T = 512 101 -> 83, T = 1000 127 -> 111.
struct SharedArgs {
    StreamArgs set[2];
    unsigned shared_blocks;              // the shared list's number of blocks, at most
};

// Reports a list that was cut for another block size.
__device__ __forceinline__ bool list_fits(int4 head, int rows, int *ctrl) {
    if (head.y == rows) return true;
    if (threadIdx.x == 0 && blockIdx.x == 0)
        __hip_atomic_fetch_or(ctrl + moe::kCtrlStatus, 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return false;
}

template <bool EVEN1, bool EVEN2, int TT, int WR>
__global__ __launch_bounds__(kThreads, TT == 2 ? 4 : 3)
void ffn_stream_shared_kernel(SharedArgs p) {
    __shared__ __attribute__((aligned(16))) char lds[kWaves * 2 * TT * MOE_WAVE * 16];
    __shared__ int s_ok;
    // The arguments by set, without a copy: a load from the kernel's argument segment with a computed offset.
    const StreamArgs *sets = (const StreamArgs *)__builtin_amdgcn_kernarg_segment_ptr();
    const unsigned id = blockIdx.x, n1s = p.shared_blocks * p.set[1].s[0].tiles_pad;
    const bool first = id < n1s;                                     // of the shared expert's first stage
    const unsigned item1 = first ? p.set[1].s[0].pad_div(id) : p.set[0].s[0].pad_div(id - n1s);
    const unsigned guess = 1 + item1, last = first ? p.set[1].list_last : p.set[0].list_last;
    const int4 head_r = load_const(p.set[0].blocks, 0), head_s = load_const(p.set[1].blocks, 0);
    const int4 ent1 = load_const(first ? p.set[1].blocks : p.set[0].blocks, guess < last ? guess : last);
    const int min_r = load_const(p.set[0].ctrl, 0).w, min_s = load_const(p.set[1].ctrl, 0).w;
    asm volatile("" ::"s"(head_r.x), "s"(head_s.x), "s"(ent1.x), "s"(ent1.y), "s"(ent1.z), "s"(ent1.w), "s"(min_r), "s"(min_s));
    const bool ok_r = list_fits(head_r, TT * 16, p.set[0].ctrl), ok_s = list_fits(head_s, TT * 16, p.set[1].ctrl);
    const unsigned blocks_r = ok_r ? static_cast<unsigned>(head_r.x) : 0u, blocks_s = ok_s ? static_cast<unsigned>(head_s.x) : 0u;
    const int ks1 = p.set[0].s[0].KS, ks2_r = p.set[0].s[1].KS, ks2_s = p.set[1].s[1].KS;
    const unsigned n1r = blocks_r * p.set[0].s[0].tiles_pad, n2s = blocks_s * p.set[1].s[1].tiles_pad,
                   n2r = blocks_r * p.set[0].s[1].tiles_pad;
    bool shared = first;
    if (id >= n1s + n1r) shared = id - (n1s + n1r) < n2s;
    const StreamArgs &a = sets[shared ? 1 : 0];
    // the routed slots are cut as in a launch of their own; the shared slot's chain may also hide behind the routed stream
    const int wide = shared ? wide_on(head_s, (p.set[1].s[0].tiles + kWaves - 1) / kWaves, min_s, ks1, ks2_s, stream_ns(blocks_r, ks1, ks2_r))
                            : wide_on(head_r, (p.set[0].s[0].tiles + kWaves - 1) / kWaves, min_r, ks1, ks2_r);
    const WideBlocks n = {shared ? head_s.x + static_cast<int>(blocks_r) : head_r.x, shared ? head_s.z : head_r.z};
    if (id < n1s + n1r) {
        if (item1 >= (first ? blocks_s : blocks_r)) return;
        const unsigned tile = (first ? id : id - n1s) - item1 * a.s[0].tiles_pad;
        run_item<true, EVEN1, TT, WR>(a, a.s[0], lds, &s_ok, wide, n, item1, tile, ent1);
    } else {
        const unsigned id2 = id - (n1s + n1r) - (shared ? 0 : n2s);
        if (!shared && id2 >= n2r) return;
        const unsigned item = a.s[1].pad_div(id2);
        run_item<false, EVEN2, TT, WR>(a, a.s[1], lds, &s_ok, wide, n, item, id2 - item * a.s[1].tiles_pad, load_const(a.blocks, 1 + item));
    }
}

template <bool L1, bool L2>
void launch_shared(const SharedArgs &p, int block_rows, unsigned blocks, hipStream_t st) {
    if (block_rows == 32) hipLaunchKernelGGL((ffn_stream_shared_kernel<L1, L2, 2, 64>), dim3(blocks), dim3(kThreads), 0, st, p);
    else hipLaunchKernelGGL((ffn_stream_shared_kernel<L1, L2, 4, 64>), dim3(blocks), dim3(kThreads), 0, st, p);
}

// ---------------------------------------------------------------------------------------------
// Batches that ffn_is_big() takes: every slot with more than kWideMin requests as wide blocks of two packed tiles a
// wavefront, the others as streaming items (one block each), in one launch of two workgroups a CU with the registers for both.
// The blocks are looked up in the list by their number among the wide or the streaming ones (find_entry), not by their place in it: a wide
// block has as many ids as it has groups of tiles, and only a slot can have a streaming block, so the worst-case grid stays small (32000 workgroups at T = 8192, k = 8, C = 16,
// d_h = 4096, d_e = 1536, where ids for every tile of every block of 64 rows would be 166000) and no workgroup has to walk a list.
// Wide blocks come first: their chains are the longest and hide behind the streams.  Against blocks of 128 rows x four tiles in two
// launches of their own before the streaming launch, us of these launches, least and most of five inputs: T = 8192, d_h = 4096,
// d_e = 1536 180 and 645 -> 148 and 536, T = 3000 127 and 164 -> 108 and 141; d_h = 2048, d_e = 1408, T = 3000 77 and 207 -> 63 and 148;
// d_e = 768, T = 4000 57 and 181 -> 50 and 114.  Slower where nearly nothing is wide, the slots are many and ffn_is_big() cannot tell (128
// slots of 64 rows, T*k = 128*C, d_h = 2048, d_e = 768 304 -> 309; 199 of 40 rows and one of 300, T*k = 82*C, d_h = 7168, d_e = 256
// 655 -> 737), and where a few blocks are all there is (one slot of 500 rows, d_h = d_e = 2048 35 -> 39).
struct BigArgs {
    StreamArgs a;
    int groups[2];                       // workgroups of a wide block: groups of eight packed tiles of a stage
    FastDiv group_div[2];                // division by groups
    int groups_sum, pads_sum;            // groups and tiles_pad of both stages together
};

// Blocks of 128 rows from this many first-stage workgroups of them on, else of 64 rows (us, blocks of 128 and of 64 rows:
// 192 such workgroups, d_h = 2048, d_e = 768 79 and 94; 240, d_h = 4096, d_e = 1536 207 and 220; 360 248 and 290; but 154, d_h = 2048,
// d_e = 1408 108 and 98; 120, d_h = 4096 178 and 169; 36 168 and 144)
constexpr int kBigMinWorkgroups = 176;
constexpr int kBigMaxCut = 8;            // blocks of 64 rows of slots with more than kWideMin requests that may be streaming items

struct BigItem { int4 ent; int index; };   // an entry of the work list and its place in it; index -1: none
// The r-th entry of a list of n that is a streaming block (a slot with at most `cut` requests) or, `wide`, that leads a block of
// wr rows (64 or 128) of a slot with more.  A slot's entries are neighbours.  Uniform over the wavefront.  Lists of up to 512 blocks
// are one round trip; the 1000 blocks of a batch that is local as a whole are two, of a launch of several hundred microseconds.
__device__ __forceinline__ BigItem find_entry(const int32_t *blocks, int n, bool wide, int cut, int wr, int r, int lane) {
    constexpr int kGroups = 8;                                       // groups of 64 entries that are requested at once
    const int4 *list = reinterpret_cast<const int4 *>(blocks) + 1;
    for (int j0 = 0; j0 < n; j0 += kGroups * MOE_WAVE) {
        int4 e[kGroups];
#pragma unroll
        for (int q = 0; q < kGroups; ++q) {
            const int g0 = j0 + q * MOE_WAVE, j = g0 + lane;
            e[q] = make_int4(0, 0, 0, 0);
            if (g0 < n) e[q] = list[j < n ? j : n - 1];
        }
#pragma unroll
        for (int q = 0; q < kGroups; ++q) {
            const int g0 = j0 + q * MOE_WAVE;
            if (g0 >= n) break;
            const bool over = e[q].z - e[q].w > cut;
            const bool mine = g0 + lane < n && over == wide && (!wide || ((e[q].y - e[q].w) & (wr - 1)) == 0);
            const unsigned long long m = __ballot(mine);
            const int count = __popcll(m);
            if (r < count) {
                const int before = __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(m >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), 0));
                const int src = __builtin_ctzll(__ballot(mine && before == r));
                return {make_int4(__builtin_amdgcn_readlane(e[q].x, src), __builtin_amdgcn_readlane(e[q].y, src),
                                  __builtin_amdgcn_readlane(e[q].z, src), __builtin_amdgcn_readlane(e[q].w, src)), g0 + src};
            }
            r -= count;
        }
    }
    return {make_int4(0, 0, 0, 0), -1};
}

// A 64-row block of a wide slot as streaming items after all (a caller's threshold says so): eight tiles of it one after the other by one
// workgroup, since the grid has no ids for every tile.  One kind of item per stage, for a full block.
template <bool STAGE1, bool EVEN>
__device__ __forceinline__ void run_untiled(const StreamArgs &a, const StageArgs &g_, char *lds, int *s_ok, int item, int group, int slot,
                                            int row0, int row_end) {
    constexpr int TT = 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / MOE_WAVE), lane = threadIdx.x % MOE_WAVE;
    const int t0 = group * 2 * kWaves, t1 = t0 + 2 * kWaves < g_.tiles ? t0 + 2 * kWaves : g_.tiles;
#pragma unroll 1
    for (int tile = t0; tile < t1; ++tile) {
        StageArgs g = g_;                                            // opaque copies, as in the loop over a long list
        asm volatile("" : "+s"(g.KS), "+s"(g.tiles));
        if (tile > t0) __syncthreads();                              // the LDS buffer is reused
        const char *w = g.Wp + (static_cast<size_t>(slot) * g.tiles + tile) * g.KS * 2048;
        if constexpr (STAGE1) {
            stream_item_lines<8, TT, false, EVEN>(a, g, lds, w, tile, row0, row_end, wave, lane);
            __syncthreads();
            store_act<TT>(a, lds, TT, item, tile, row0, row_end);
            announce_tiles(a, item, g.tiles);
        } else if (stream_item_down<4, TT, 1, false, 1>(a, g, lds, s_ok, w, 0, item, tile, g.tiles, wave, lane)) {
            __syncthreads();
            store_rows<TT>(a, g, lds, 2, 4, tile, row0, row_end);
        } else {
            store_nan_rows(a, g, tile, row0, row_end - row0 < TT * 16 ? row_end - row0 : TT * 16);
        }
    }
}

// n_blocks: entries of the list; n_wide: blocks of the wide slots; id: of the stage's wide or streaming ids.  A block is named by its
// first entry of the list: that entry's control lines and, with 128 rows, the `act` of that entry and the next.
template <bool STAGE1, bool EVEN>
__device__ __forceinline__ void run_big(const BigArgs &p, char *lds, int *s_ok, bool wide, int cut, bool tiled, bool rows128,
                                        int n_blocks, int n_wide, unsigned id) {
    const StreamArgs &a = p.a;
    const StageArgs &g = a.s[STAGE1 ? 0 : 1];
    const int groups = p.groups[STAGE1 ? 0 : 1];
    int b = static_cast<int>(g.pad_div(id)), r = b;                  // streaming: block, and tile below
    if (wide) {
        // Ids go round-robin over the eight XCDs; each takes an eighth of the wide items as one run, a slot's items block-fastest:
        // the blocks of one group of tiles start next to each other on one XCD and share the expert's tiles in that L2, and the
        // XCD needs the rows and weights of few slots.
        const int n = n_wide * groups, x = id & 7, each = n >> 3, more = n & 7, place = static_cast<int>(id >> 3);
        if (place >= each + (x < more ? 1 : 0)) return;
        b = x * each + (x < more ? x : more) + place;
        r = static_cast<int>(p.group_div[STAGE1 ? 0 : 1](b));        // a slot of nb blocks has nb * groups items: its block r has the slot of item b
    }
    const int shift = rows128 ? 7 : 6, wr = 1 << shift;              // rows of a wide block
    const BigItem it = find_entry(a.blocks, n_blocks, wide, cut, wr, r, moe::lane_id());
    if (it.index < 0) return;
    const int lo = it.ent.w, hi = it.ent.z;
    if (!wide) {
        run_stream_item<STAGE1, EVEN, 4>(a, g, lds, s_ok, it.index, static_cast<int>(id) - b * g.tiles_pad, it.ent);
        return;
    }
    const int nb = (hi - lo + wr - 1) >> shift, nth = (it.ent.y - lo) >> shift, at = b - (r - nth) * groups, group = at / nb, block = at % nb;
    const int row0 = lo + block * wr, m = hi - row0 < wr ? hi - row0 : wr;
    const int item = it.index + ((block - nth) << (shift - 6));
    if (!tiled) run_untiled<STAGE1, EVEN>(a, g, lds, s_ok, item, group, it.ent.x, row0, hi);
    else if (m > 64) wide_item2<STAGE1, 8>(a, g, lds, s_ok, item, group, groups, it.ent.x, row0, m);
    else wide_item2<STAGE1, 4>(a, g, lds, s_ok, item, group, groups, it.ent.x, row0, m);
}

template <bool EVEN1, bool EVEN2>
__global__ __launch_bounds__(kThreads, 2)
void ffn_big_kernel(BigArgs p) {
    __shared__ __attribute__((aligned(16))) char lds[kWaves * 2 * 4 * MOE_WAVE * 16];
    static_assert(2 * 128 * 128 <= sizeof(lds), "the two token tiles of a wide block must fit");
    __shared__ int s_ok;
    const int4 head = load_const(p.a.blocks, 0);
    const int wide_min = load_const(p.a.ctrl, 0).w;
    if (!list_fits(head, 64, p.a.ctrl)) return;
    // The surplus of the worst-case grid leaves before anything else is worked out (30000 workgroups at T = 8192, d_h = 4096, d_e = 1536: a layer
    // with 36 blocks 152.9 us without this line, 148.7 with it).
    if (blockIdx.x >= 16u + head.z * p.groups_sum + (head.x - head.z + kBigMaxCut) * p.pads_sum) return;
    // a caller's threshold: as in the other launches for blocks of 64 rows, the same for blocks of 128, which it takes before them
    const int groups64 = (p.a.s[0].tiles + kWaves - 1) / kWaves;
    const bool rows128 = wide_min > 0 ? head.w * groups64 >= wide_min : head.w * p.groups[0] >= kBigMinWorkgroups;
    // a few blocks that nothing hides are cut into streaming items as in the other launches (wide_on)
    const bool tiled = wide_min > 0 ? head.z * groups64 >= wide_min
                                    : head.z > kBigMaxCut || wide_on(head, groups64, 0, p.a.s[0].KS, p.a.s[1].KS);
    const bool any = tiled || head.z > kBigMaxCut;                   // ids of their own for the wide slots' blocks
    const int cut = any ? kWideMin : 0x7fffffff;
    const int n_wide = any ? (rows128 ? head.w : head.z) : 0;
    const unsigned n_stream = head.x - (any ? head.z : 0);
    unsigned id = blockIdx.x;
    const unsigned w1 = (n_wide * p.groups[0] + 7u) & ~7u, s1 = n_stream * p.a.s[0].tiles_pad;
    if (id < w1 + s1) {
        const bool wide = id < w1;
        run_big<true, EVEN1>(p, lds, &s_ok, wide, cut, tiled, rows128, head.x, n_wide, wide ? id : id - w1);
        return;
    }
    id -= w1 + s1;
    const unsigned w2 = (n_wide * p.groups[1] + 7u) & ~7u, s2 = n_stream * p.a.s[1].tiles_pad;
    if (id < w2 + s2) {
        const bool wide = id < w2;
        run_big<false, EVEN2>(p, lds, &s_ok, wide, cut, tiled, rows128, head.x, n_wide, wide ? id : id - w2);
    }
}

template <bool L1, bool L2, bool WRAP>
void launch(const StreamArgs &a, int block_rows, unsigned blocks, hipStream_t st) {
    if (block_rows == 32) hipLaunchKernelGGL((ffn_stream_kernel<L1, L2, 2, 64, WRAP>), dim3(blocks), dim3(kThreads), 0, st, a);
    else hipLaunchKernelGGL((ffn_stream_kernel<L1, L2, 4, 64, WRAP>), dim3(blocks), dim3(kThreads), 0, st, a);
}

template <bool WRAP>
void launch_even(const StreamArgs &a, int block_rows, unsigned blocks, hipStream_t st) {
    const bool l1 = a.s[0].KS % 2 == 0, l2 = a.s[1].KS % 2 == 0;
    if (l1 && l2) launch<true, true, WRAP>(a, block_rows, blocks, st);
    else if (l1) launch<true, false, WRAP>(a, block_rows, blocks, st);
    else if (l2) launch<false, true, WRAP>(a, block_rows, blocks, st);
    else launch<false, false, WRAP>(a, block_rows, blocks, st);
}

StreamArgs stream_args(const moe::FfnCall &c, int T, int d_h) {
    const int block_rows = moe::ffn_block_rows(T);
    StreamArgs a;
    a.blocks = c.blocks; a.perm = c.perm; a.act = c.act; a.Yp = c.Yp; a.ctrl = c.ctrl; a.k_div = fast_div(c.k);
    a.list_last = static_cast<unsigned>(moe::ffn_max_blocks(T, c.k, c.C));
    a.spin_limit = 1 << 20;
    a.act_block_bytes = static_cast<uint32_t>(moe::ffn_act_block_bytes(T, c.d_e));
    a.s[0].B = static_cast<const uint16_t *>(c.X);
    a.s[0].Wp = static_cast<const char *>(c.W13p);
    a.s[0].tiles = c.d_e / 16; a.s[0].KS = d_h / 32; a.s[0].b_stride = d_h; a.s[0].out_stride = 0;
    a.s[1].B = c.act;
    a.s[1].Wp = static_cast<const char *>(c.W2p);
    a.s[1].tiles = d_h / 32; a.s[1].KS = c.d_e / 32; a.s[1].b_stride = 0; a.s[1].out_stride = d_h;
    a.s[0].items = a.s[0].tiles;
    a.s[1].items = block_rows == 32 ? a.s[1].tiles : (a.s[1].tiles + 1) / 2;   // 64-row launch: a stage-2 workgroup owns a pair of tiles
    for (int i = 0; i < 2; ++i) {
        a.s[i].tiles_pad = (a.s[i].items + 7) / 8 * 8;
        a.s[i].pad_div = fast_div(a.s[i].tiles_pad);
    }
    return a;
}

}  // namespace

namespace moe {

int launch_ffn_stream(const FfnCall &c, int T, int d_h, hipStream_t st) {
    const long long items = ffn_max_blocks(T, c.k, c.C);
    if (items > kMaxItems) return MOE_ESHAPE;
    const StreamArgs a = stream_args(c, T, d_h);
    if (ffn_is_big(T, c.k, c.C, d_h, c.d_e)) {
        BigArgs p;
        p.a = a;
        for (int i = 0; i < 2; ++i) {
            p.groups[i] = (a.s[i].tiles + 2 * kWaves - 1) / (2 * kWaves);
            p.group_div[i] = fast_div(p.groups[i]);
        }
        p.groups_sum = p.groups[0] + p.groups[1];
        p.pads_sum = a.s[0].tiles_pad + a.s[1].tiles_pad;
        if (items * p.groups[0] > 0x7fffffffLL || items * p.groups[1] > 0x7fffffffLL) return MOE_ESHAPE;
        const long long grid = items * p.groups_sum + 16 + static_cast<long long>(c.C + kBigMaxCut) * p.pads_sum;
        if (grid > 0x7fffffffLL) return MOE_ESHAPE;
        const bool l1 = a.s[0].KS % 2 == 0, l2 = a.s[1].KS % 2 == 0;
        const dim3 blocks(static_cast<unsigned>(grid)), threads(kThreads);
        if (l1 && l2) hipLaunchKernelGGL((ffn_big_kernel<true, true>), blocks, threads, 0, st, p);
        else if (l1) hipLaunchKernelGGL((ffn_big_kernel<true, false>), blocks, threads, 0, st, p);
        else if (l2) hipLaunchKernelGGL((ffn_big_kernel<false, true>), blocks, threads, 0, st, p);
        else hipLaunchKernelGGL((ffn_big_kernel<false, false>), blocks, threads, 0, st, p);
        return MOE_OK;
    }
    const long long lanes = items < kFfnLaneBlocks ? items : kFfnLaneBlocks;
    const long long n1 = lanes * a.s[0].tiles_pad, n2 = lanes * a.s[1].tiles_pad;
    if (n1 + n2 > 0x7fffffffLL) return MOE_ESHAPE;
    // only a batch whose list can be longer than the lanes needs the code that walks it
    if (items > kFfnLaneBlocks) launch_even<true>(a, ffn_block_rows(T), static_cast<unsigned>(n1 + n2), st);
    else launch_even<false>(a, ffn_block_rows(T), static_cast<unsigned>(n1 + n2), st);
    return MOE_OK;
}

// Routed blocks that the launch of two sets has workgroups for.  It has no loop over a long list, and the surplus of its grid
// costs more the larger the bound is (us a step with the shared expert, two launches and one, means of three inputs: bound 131,
// d_h = 7168, d_e = 2048, T = 380 358 and 292; 157, d_h = 2048, d_e = 1408, T = 1500 158 and 144; 195, T = 1900 179 and 168; 204,
// d_e = 768, T = 1500 104 and 93; 203, d_h = 4096, d_e = 1536, T = 1500 225 and 221; 267, d_h = 2048, d_e = 768, T = 2000 111 and 113).  A set
// that takes the launch for large batches keeps a call of its own (d_h = 7168, d_e = 2048, shared width 2048: T = 900 389, in one
// launch of streaming and 64-row items 399; T = 1500 516 and 549).
constexpr long long kSharedMaxBlocks = 224;
bool ffn_stream_takes_shared(const FfnCall &c, const FfnCall &sh, int T, int d_h) {
    const long long items = ffn_max_blocks(T, c.k, c.C), items_s = ffn_max_blocks(T, sh.k, sh.C);
    if (ffn_is_big(T, c.k, c.C, d_h, c.d_e) || ffn_is_big(T, sh.k, sh.C, d_h, sh.d_e) || items > kSharedMaxBlocks || items_s > kFfnLaneBlocks || (c.d_e / 32) % 2 != (sh.d_e / 32) % 2) return false;
    const StreamArgs r = stream_args(c, T, d_h), s = stream_args(sh, T, d_h);
    return items * (r.s[0].tiles_pad + r.s[1].tiles_pad) + items_s * (s.s[0].tiles_pad + s.s[1].tiles_pad) <= 0x7fffffffLL;
}

void launch_ffn_stream_shared(const FfnCall &c, const FfnCall &sh, int T, int d_h, hipStream_t st) {
    SharedArgs p;
    p.set[0] = stream_args(c, T, d_h);
    p.set[1] = stream_args(sh, T, d_h);
    const unsigned items = static_cast<unsigned>(ffn_max_blocks(T, c.k, c.C));
    p.shared_blocks = static_cast<unsigned>(ffn_max_blocks(T, sh.k, sh.C));
    const unsigned blocks = items * (p.set[0].s[0].tiles_pad + p.set[0].s[1].tiles_pad) +
                            p.shared_blocks * (p.set[1].s[0].tiles_pad + p.set[1].s[1].tiles_pad);
    const int block_rows = ffn_block_rows(T);
    const bool l1 = p.set[0].s[0].KS % 2 == 0, l2 = p.set[0].s[1].KS % 2 == 0;
    if (l1 && l2) launch_shared<true, true>(p, block_rows, blocks, st);
    else if (l1) launch_shared<true, false>(p, block_rows, blocks, st);
    else if (l2) launch_shared<false, true>(p, block_rows, blocks, st);
    else launch_shared<false, false>(p, block_rows, blocks, st);
}

}  // namespace moe
