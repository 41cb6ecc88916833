// a0-a4 in ONE launch: gating selection for all tokens, then Alg. 1 and this instance's
// dispatch (Janus Sec. 3.4, workflow Steps 0-4).  At decode sizes each of these steps is a few
// microseconds of work behind a launch of about the same cost, so three launches become one.
//
// Every workgroup routes 4, 8 or 16 tokens (one per wavefront; the fewer, the smaller the batch:
// launch_front) and publishes their expert ids with agent-scope stores; the workgroup that finishes last (an atomic ticket, nobody waits) then
// runs Alg. 1 and the counting sort on its own, reading the ids with agent-scope loads because
// they were written on other XCDs.
//
// The gated variants start one step earlier (Sec. 3.3: gating runs on the MoE side, from the
// complete activations): the logits are the router's linear layer X * W_r^T (+ bias), a launch of their own
// before the one that starts from logits.  (In one launch, with the workgroup that completed a token group
// routing its 16 tokens, the routing shared its CU with the products: 44 us at T = 512, E = 256, d_h = 7168
// against 25 us for the two launches, and 25 against 18 us at T = 32.)
#include "dispatch_dev.h"

namespace {

struct FrontArgs {
    const float *logits;
    int T, E, k;
    moe_route_cfg cfg;
    int32_t *ids;
    float *w;
    moe::SchedTables tb;
    int n_inst, C, n_words, g_self;
    int32_t *rid, *act_rep, *load, *slot_count, *slot_off, *perm, *pos, *blocks;
    int32_t *ticket;
    int block_rows;
    // batches too large for the one-workgroup tail (launch from logits only): the routing workgroups
    // raise the activated experts in act_bits, the last one runs Step 2 of Alg. 1 from them, and two
    // further launches (front_count_kernel, front_scatter_kernel) rewrite and sort the requests in chunks
    uint32_t *act_bits;                  // [kBitWords], zero between calls; null = one-workgroup tail
    int32_t *hist;                       // [n_chunks][C]
    int chunk_pairs, n_chunks;
    int solo;                            // one workgroup routes the batch and goes on without a ticket
    int tok_per_wave;                    // tokens such a wavefront routes one after the other
    int tok_per_wg;                      // wavefronts of a workgroup that route a token (4, 8 or 16)
};
constexpr int kBitWords = MOE_MAX_EXPERTS / 32;
constexpr int kChunkPairs = 2048;

// ------------------------------------------------------------------ the gate's linear layer
struct GateArgs {
    const uint16_t *X, *Wr;              // bf16 [T,d_h], [E,d_h]
    const float *bias;                   // [E] or null
    float *logits;                       // [T,E]
    int T, E, d_h;
    int e_tiles;                         // ceil(E/16) expert tiles
};
constexpr int kGateWaves = 16;
constexpr int kGateUnroll = 4;
constexpr int kGateDepth = 2;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Logits of TT token tiles (16 tokens each) against expert tile j (16 experts).  MFMA 16x16x32: the
// router rows are the A operand (lane l: expert l%16, 8 columns at (l/16)*8 of the K-step), the
// token rows the B operand (same shape), and the D tile leaves lane l with experts (l/16)*4..+3
// of token l%16.  Rows past T or E repeat the last valid row and are not stored.  The 16 wavefronts split the
// hidden dimension.
//
// This wavefront's share of the sum, operands read straight into the MFMA layout: every lane
// requests its own 16 bytes of its own row, four requests per 64 bytes.  Used when the hidden
// size is not a multiple of 64.
template <int TT>
__device__ __forceinline__ void gate_acc_steps(const GateArgs &a, int t0, int j, int wave, int lane, f32x4 (&acc)[TT]) {
    const int KS = a.d_h / 32;
    const int per = (KS + kGateWaves - 1) / kGateWaves;
    const int k0 = wave * per;
    const int k1 = k0 + per < KS ? k0 + per : KS;
    int e = j * 16 + (lane & 15);
    e = e < a.E ? e : a.E - 1;
    const char *wb = reinterpret_cast<const char *>(a.Wr) + (static_cast<size_t>(e) * a.d_h + (lane >> 4) * 8) * 2;
    const char *xb[TT];
#pragma unroll
    for (int t = 0; t < TT; ++t) {
        int tok = t0 + t * 16 + (lane & 15);
        tok = tok < a.T ? tok : a.T - 1;
        xb[t] = reinterpret_cast<const char *>(a.X) + (static_cast<size_t>(tok) * a.d_h + (lane >> 4) * 8) * 2;
    }
    // kGateUnroll K-steps of both operands in flight; steps past the share load the last valid step
    // again and multiply by zero, so the loop has no tail
    const bf16x8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int kk = k0; kk < k1; kk += kGateUnroll) {
        bf16x8 av[kGateUnroll], bv[kGateUnroll][TT];
#pragma unroll
        for (int u = 0; u < kGateUnroll; ++u) {
            const int q = kk + u < k1 ? kk + u : k1 - 1;
            av[u] = *reinterpret_cast<const bf16x8 *>(wb + q * 64);
#pragma unroll
            for (int t = 0; t < TT; ++t) bv[u][t] = *reinterpret_cast<const bf16x8 *>(xb[t] + q * 64);
        }
#pragma unroll
        for (int u = 0; u < kGateUnroll; ++u)
#pragma unroll
            for (int t = 0; t < TT; ++t)
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kk + u < k1 ? av[u] : zero, kk + u < k1 ? bv[u][t] : zero, acc[t], 0, 0, 0);
    }
}

// The same share with whole-line reads (hidden size a multiple of 64): a super-step is 64 columns =
// one 128-byte line of each row; a load instruction fetches 8 whole lines (lane l:
// row l/8, 16-byte chunk l%8), a quarter of the requests of the direct form, and the MFMA layout
// comes from a round trip through a wave-private LDS tile (chunks XOR-swizzled by row so
// that the row-major writes and the column-wise reads both spread over the banks).  Wavefront w
// takes super-steps w, w+16, ...; kGateDepth of them are in flight.
template <int TT>
__device__ __forceinline__ void gate_acc_lines(const GateArgs &a, int t0, int j, char *stage, int wave, int lane,
                                               f32x4 (&acc)[TT]) {
    constexpr int L = 2 + 2 * TT;                                    // load instructions per super-step
    const int SS = a.d_h / 64;
    const int n = (SS - wave + kGateWaves - 1) / kGateWaves;
    char *st = stage + wave * (L * 1024);                            // [router rows | token rows][16 rows][128 bytes]
    const char *p[L];
#pragma unroll
    for (int h = 0; h < L; ++h) {
        const int r = h * 8 + (lane >> 3);                           // row of the 16 router + TT*16 token rows
        if (h < 2) {
            int e = j * 16 + r;
            e = e < a.E ? e : a.E - 1;
            p[h] = reinterpret_cast<const char *>(a.Wr) + static_cast<size_t>(e) * a.d_h * 2 + (lane & 7) * 16;
        } else {
            int t = t0 + r - 16;
            t = t < a.T ? t : a.T - 1;
            p[h] = reinterpret_cast<const char *>(a.X) + static_cast<size_t>(t) * a.d_h * 2 + (lane & 7) * 16;
        }
    }
    // LDS: row R of an operand at R*128, its 16-byte chunk c at ((c ^ (R & 7)) * 16)
    const uint32_t wr_lds = ((lane >> 3) * 128) + (((lane & 7) ^ (lane >> 3)) * 16);
    const uint32_t rd_row = (lane & 15) * 128, rd_sw = lane & 7, rd_g = lane >> 4;
    bf16x8 ld[kGateDepth][L];
#define MOE_GATE_LOAD(d, i)                                                                      \
    do {                                                                                         \
        const size_t off_ = static_cast<size_t>(wave + kGateWaves * (i)) * 128;                  \
        _Pragma("unroll") for (int q = 0; q < L; ++q)                                            \
            ld[d][q] = *reinterpret_cast<const bf16x8 *>(p[q] + off_);                           \
    } while (0)
#pragma unroll
    for (int d = 0; d < kGateDepth; ++d)
        if (d < n) MOE_GATE_LOAD(d, d);
    for (int i = 0; i < n; i += kGateDepth) {
#pragma unroll
        for (int d = 0; d < kGateDepth; ++d) {
            if (i + d < n) {                                         // wave-uniform
#pragma unroll
                for (int q = 0; q < L; ++q) *reinterpret_cast<bf16x8 *>(st + q * 1024 + wr_lds) = ld[d][q];
                asm volatile("" ::: "memory");
                if (i + d + kGateDepth < n) MOE_GATE_LOAD(d, i + d + kGateDepth);
#pragma unroll
                for (int ss = 0; ss < 2; ++ss) {
                    const uint32_t o = rd_row + (((4 * ss + rd_g) ^ rd_sw) * 16);
                    const bf16x8 av = *reinterpret_cast<const bf16x8 *>(st + o);
#pragma unroll
                    for (int t = 0; t < TT; ++t) {
                        const bf16x8 bv = *reinterpret_cast<const bf16x8 *>(st + (1 + t) * 2048 + o);
                        acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv, acc[t], 0, 0, 0);
                    }
                }
                asm volatile("" ::: "memory");
            }
        }
    }
#undef MOE_GATE_LOAD
}

// A workgroup computes TT*16 tokens x 16 experts.  The partial tiles of the 16 wavefronts are summed in
// wavefront order, so results are reproducible and do not depend on TT.
// Workgroups go to the 8 XCDs round-robin: the XCDs form a grid of 4 token shares x 2 expert shares, so each L2 reads
// a quarter of the activations and half of the router matrix.
// Bound by the operand tiles on their way through the L1s (176 MB at T = 512, E = 256, d_h = 7168).  11.7 us there;
// with four super-steps in flight 15.6 us (the register file spills), with three 12.5 us, with tiles of 16 x 16
// 16.1 us.
template <int TT, bool LINES>
__global__ __launch_bounds__(kGateWaves * MOE_WAVE)
void gate_kernel(GateArgs a) {
    // staging tiles of the line form, then the partial tiles
    __shared__ __attribute__((aligned(16))) char lds[kGateWaves * (LINES ? 2 + 2 * TT : TT) * 1024];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / MOE_WAVE), lane = moe::lane_id();
    const int r = blockIdx.x / 8, xcd = blockIdx.x % 8, eh = (a.e_tiles + 1) / 2;
    const int tg = xcd % 4 + 4 * (r / eh), j = r % eh + (xcd / 4) * eh;
    if (j >= a.e_tiles) return;
    const int t0 = tg * (TT * 16);
    if (t0 >= a.T) return;
    // the bias of this lane's four experts, fetched up front
    float bias[4] = {0.f, 0.f, 0.f, 0.f};
    if (a.bias && wave < TT) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int ee = j * 16 + (lane >> 4) * 4 + i;
            bias[i] = a.bias[ee < a.E ? ee : a.E - 1];
        }
    }
    f32x4 acc[TT];
#pragma unroll
    for (int t = 0; t < TT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    if constexpr (LINES) {
        gate_acc_lines<TT>(a, t0, j, lds, wave, lane, acc);
        __syncthreads();                                             // the staging tiles give way to the partial tiles
    } else {
        gate_acc_steps<TT>(a, t0, j, wave, lane, acc);
    }
    f32x4 *part = reinterpret_cast<f32x4 *>(lds);
#pragma unroll
    for (int t = 0; t < TT; ++t) part[(t * kGateWaves + wave) * MOE_WAVE + lane] = acc[t];
    __syncthreads();
    if (wave < TT) {
        const f32x4 *mine = part + wave * kGateWaves * MOE_WAVE + lane;
        f32x4 s = mine[0];
#pragma unroll
        for (int w = 1; w < kGateWaves; ++w) s += mine[w * MOE_WAVE];
        const int t = t0 + wave * 16 + (lane & 15);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int ee = j * 16 + (lane >> 4) * 4 + i;
            if (t < a.T && ee < a.E) a.logits[static_cast<size_t>(t) * a.E + ee] = s[i] + bias[i];
        }
    }
}

// Tiles of 32 tokens read a quarter less than tiles of 16 (48 rows for 2 x 16 logits a lane instead of 64), and are
// taken when they still give every CU a workgroup.
constexpr long long kGateWideTiles = 256;
int launch_gate(const void *X, const void *Wr, const float *bias, float *logits, int T, int E, int d_h, hipStream_t st) {
    GateArgs a;
    a.X = static_cast<const uint16_t *>(X); a.Wr = static_cast<const uint16_t *>(Wr); a.bias = bias; a.logits = logits;
    a.T = T; a.E = E; a.d_h = d_h; a.e_tiles = (E + 15) / 16;
    const bool lines = d_h % 64 == 0;
    const bool wide = static_cast<long long>((T + 31) / 32) * a.e_tiles >= kGateWideTiles;
    const int groups = wide ? (T + 31) / 32 : (T + 15) / 16;
    const long long blocks = static_cast<long long>((groups + 3) / 4) * 8 * ((a.e_tiles + 1) / 2);
    if (blocks > 0x7fffffffLL) return MOE_ESHAPE;
    const dim3 grid(static_cast<unsigned>(blocks)), threads(kGateWaves * MOE_WAVE);
    if (wide && lines) hipLaunchKernelGGL((gate_kernel<2, true>), grid, threads, 0, st, a);
    else if (wide) hipLaunchKernelGGL((gate_kernel<2, false>), grid, threads, 0, st, a);
    else if (lines) hipLaunchKernelGGL((gate_kernel<1, true>), grid, threads, 0, st, a);
    else hipLaunchKernelGGL((gate_kernel<1, false>), grid, threads, 0, st, a);
    return MOE_OK;
}

// ------------------------------------------------------------------ selection, Alg. 1 and dispatch
// Decode-size tail (up to kRegPairs requests): Alg. 1 and the counting sort with every request id
// held in registers.  Wavefront w owns requests [w*gpw*64, (w+1)*gpw*64), the mapping the sort needs,
// so the ids are read from memory exactly once and everything after that runs out of LDS and registers.
constexpr int kGpwMax = 8;                                            // 64-request groups per wavefront (1 and 2: front_tail_few; 4 and 8: front_tail_small)
constexpr int kRegPairs = moe::kFrontWaves * kGpwMax * MOE_WAVE;      // 8192
constexpr int kFewPairs = 2 * moe::kFrontWaves * MOE_WAVE;            // 2048: up to two requests a thread
constexpr int kSlotOfLds = 8192;                                      // E*n_inst entries of slot_of kept in LDS
// A batch of a few tokens is routed by one workgroup: the ids stay in LDS, and the publication, the ticket and the
// read-back (0.3 + 0.45 + 0.9 us at T = 8) fall away.  Its wavefronts take turns on the four SIMDs, so each further four
// tokens add a selection to the chain, and the line falls with the selection's length, about E * k
// (one workgroup against several, us: E = 64, k = 6, T = 12 5.7 and 5.9; E = 128, k = 8, T = 8 6.35 and 6.7; E = 512, k = 8, T = 8 9.3 and 9.75,
// T = 12 level; E = 1000, k = 8, T = 8 12.6 and 13.2; E = 1024, k = 32, T = 4 21.9 and 22.6, T = 16 34.5 and 23.7).  With 9 to 12 tokens and
// E * k from 768 to 2048 several would take 1 to 6 % less (E = 128, k = 8, T = 12 6.9 and 6.7; E = 256 with groups, k = 8, T = 9 9.4 and 8.8),
// but one workgroup leaves the ticket alone there, which callers with several streams have been able to rely on.
constexpr int kSoloTokens = 12;
int solo_tokens(int E, int k) { return E * k <= 2048 ? kSoloTokens : E * k <= 8192 ? 8 : 4; }

struct SmallShared {
    moe::SchedShared sched;
    moe::PermShared perm;
    alignas(16) int16_t slot_of[kSlotOfLds];
    int16_t expert_of[MOE_MAX_SLOTS];                                 // of this instance's slots; unspecified where a slot is empty
};

// The tail's layout tables in LDS, its flags and counters cleared.  Every workgroup prepares this while
// its tokens are being routed, although only the last one uses it: nothing of it follows the ticket then.
// Elements are dealt from the highest thread down, because the lowest wavefronts are the ones that route.
struct TablePrefetch {
    uint64_t host_mask, multi_mask, single_mask;
    int32_t single_rid;
    uint4 slot_of;                                                    // 8 int16 entries
};

__device__ __forceinline__ TablePrefetch prefetch_tables(const FrontArgs &a) {
    TablePrefetch t{};
    const int i = moe::kFrontThreads - 1 - threadIdx.x;
    if (i < a.E) { t.host_mask = a.tb.host_mask[i]; t.single_rid = a.tb.single_rid[i]; }
    if (i < a.n_words) t.multi_mask = a.tb.multi_mask[i];
    if (i < a.n_inst * a.n_words) t.single_mask = a.tb.single_mask[i];
    // the table is padded to a multiple of 256 bytes, so the last 16-byte read stays inside it
    if (i * 8 < a.E * a.n_inst) t.slot_of = reinterpret_cast<const uint4 *>(a.tb.slot_of)[i];
    return t;
}

// E, n_words, n_inst*n_words <= 1024 threads and E*n_inst <= 8*1024: one element each
__device__ __forceinline__ void stage_small(const FrontArgs &a, SmallShared &sh, const TablePrefetch &t) {
    const int i = moe::kFrontThreads - 1 - threadIdx.x;
    if (i < a.E) {
        sh.sched.flag[i] = 0u;
        sh.sched.host_mask[i] = t.host_mask;
        sh.sched.single_rid[i] = t.single_rid;
    }
    if (i < a.n_words) sh.sched.multi_mask[i] = t.multi_mask;
    if (i < a.n_inst * a.n_words) sh.sched.single_mask[i] = t.single_mask;
    if (i * 8 < a.E * a.n_inst) reinterpret_cast<uint4 *>(sh.slot_of)[i] = t.slot_of;
    static_assert(sizeof(sh.perm.cnt) == moe::kFrontThreads * 16, "one 16-byte store per thread clears the counters");
    reinterpret_cast<uint4 *>(&sh.perm.cnt[0][0])[i] = make_uint4(0u, 0u, 0u, 0u);
}

// VPL >= n_words; GPW >= 64-request groups per wavefront.  The request ids were written by other workgroups and are read with
// agent-scope loads.
template <int VPL, int GPW>
__device__ __forceinline__ void front_tail_small(const FrontArgs &a, SmallShared &sh, int n_pairs) {
    const int tid = threadIdx.x;
    const int wave = tid / MOE_WAVE, lane = tid % MOE_WAVE;
    const int E = a.E, n_inst = a.n_inst, C = a.C;
    const int n_groups = (n_pairs + MOE_WAVE - 1) / MOE_WAVE;
    const int gpw = (n_groups + moe::kFrontWaves - 1) / moe::kFrontWaves;   // <= GPW

    int id[GPW];
#pragma unroll
    for (int g = 0; g < GPW; ++g) {
        const int p = (wave * gpw + g) * MOE_WAVE + lane;
        id[g] = -1;
        if (g < gpw && p < n_pairs)
            id[g] = __hip_atomic_load(a.ids + p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // ---- Step 1
#pragma unroll
    for (int g = 0; g < GPW; ++g)
        if (id[g] >= 0) sh.sched.flag[id[g]] = 1u;
    __syncthreads();

    // ---- Step 2 (first wavefront), slot_of in LDS
    if (tid < MOE_WAVE) {
        const auto rep_of = [&](int e, int g) {
            const int single = sh.sched.single_rid[e], multi = (g < 0 ? 0 : g) * C + sh.slot_of[e * n_inst + (g < 0 ? 0 : g)];
            return g >= 0 ? multi : single;
        };
        const int load = moe::aebs_select_wave<VPL, VPL>(sh.sched.flag, sh.sched.host_mask, sh.sched.multi_mask,
                                                    sh.sched.single_mask, E, n_inst, a.n_words, lane, rep_of, sh.sched.rep,
                                                    a.act_rep);
        if (lane < n_inst) a.load[lane] = load;
    }
    __syncthreads();

    // ---- Step 3 and pass A of the sort
    const int rid_lo = a.g_self * C;
    int sl[GPW];                                                  // local slot, or -1
#pragma unroll
    for (int g = 0; g < GPW; ++g) {
        sl[g] = -1;
        if (id[g] >= 0) {
            const int r = sh.sched.rep[id[g]];
            a.rid[(wave * gpw + g) * MOE_WAVE + lane] = r;
            const int s = r - rid_lo;
            if (s >= 0 && s < C) { sl[g] = s; atomicAdd(&sh.perm.cnt[wave][s], 1); }
        }
    }
    __syncthreads();
    for (int s = tid; s < C; s += moe::kFrontThreads) {
        int run = 0;
#pragma unroll
        for (int w = 0; w < moe::kFrontWaves; ++w) {
            const int c = sh.perm.cnt[w][s];
            sh.perm.cnt[w][s] = run;
            run += c;
        }
        sh.perm.total[s] = run;
        a.slot_count[s] = run;
    }
    __syncthreads();
    if (wave == 0) moe::scan_slots(sh.perm, C, a.block_rows, a.slot_off, lane);
    __syncthreads();
    moe::list_blocks(sh.perm, C, a.block_rows, a.blocks);

    // ---- pass B
    if (C <= MOE_WAVE) {
        // the wavefront's running base of slot s lives in lane s: the loop over a group's slots reads
        // and bumps it with scalar-indexed lane accesses, no LDS round trip per slot
        int base_reg = lane < C ? sh.perm.cnt[wave][lane] + sh.perm.off[lane] : 0;
#pragma unroll
        for (int g = 0; g < GPW; ++g) {
            if (g < gpw) {                                            // wave-uniform
                const int p = (wave * gpw + g) * MOE_WAVE + lane;
                const int s = sl[g];
                const bool local = s >= 0;
                int row = -1;
                uint64_t todo = __ballot(local);
                while (todo) {
                    const int lead = __builtin_ctzll(todo);
                    const int s0 = __builtin_amdgcn_readlane(s, lead);
                    const uint64_t same = __ballot(local && s == s0);
                    const int b = __builtin_amdgcn_readlane(base_reg, s0);
                    if (local && s == s0) row = b + __popcll(same & moe::lanemask_lt());
                    if (lane == s0) base_reg += __popcll(same);
                    todo &= ~same;
                }
                if (p < n_pairs) {
                    a.pos[p] = row;
                    if (local) a.perm[row] = p;
                }
            }
        }
        return;
    }
    volatile int *base = &sh.perm.cnt[wave][0];
#pragma unroll
    for (int g = 0; g < GPW; ++g) {
        if (g < gpw) {                                                // wave-uniform
            const int p = (wave * gpw + g) * MOE_WAVE + lane;
            const int s = sl[g];
            const bool local = s >= 0;
            int row = -1;
            uint64_t todo = __ballot(local);
            while (todo) {
                const int lead = __builtin_ctzll(todo);
                const int s0 = __builtin_amdgcn_readlane(s, lead);
                const uint64_t same = __ballot(local && s == s0);
                const int b = base[s0] + sh.perm.off[s0];
                if (local && s == s0) row = b + __popcll(same & moe::lanemask_lt());
                __builtin_amdgcn_wave_barrier();
                if (lane == lead) base[s0] += __popcll(same);
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                todo &= ~same;
            }
            if (p < n_pairs) {
                a.pos[p] = row;
                if (local) a.perm[row] = p;
            }
        }
    }
}

// What a wavefront's lanes did to LDS before this comes before what they do after it.  The lanes run in step, but the compiler orders only
// each lane's own accesses.
__device__ __forceinline__ void wave_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The tail of batches with one or two requests a thread (GPW).  An expert has at most one slot on this instance, so which of its slots a
// request would go to and the request's place there do not wait for Alg. 1: they are worked out with Step 1, and the counts' prefix over
// the wavefronts beside Step 2; what follows Step 2 is the scan over the slots that it kept, on the second wavefront beside the stores of
// Step 3, and the stores.  Bound by the instructions of its 16 wavefronts, four to a SIMD of one CU.  Against front_tail_small, which has two
// passes over the requests and two more barriers behind Step 2, both in a kernel with all tails, us, this launch alone: E = 128, k = 8, T = 8
// 6.45 -> 6.3, T = 128 7.8 -> 7.3, T = 256 8.3 -> 8.15; E = 256, k = 8, T = 256 9.35 -> 8.9 (with groups of experts 10.9 and 10.9, T = 160 10.55
// and 10.65); E = 64, k = 6, T = 341 8.2 -> 7.7.  With four and more requests a thread the ranks ahead of
// Step 2 take what they save behind it (E = 256, k = 8, T = 512 behind the gate 23.5 and 23.7 us), so those batches keep front_tail_small.
// ids_lds: the batch's request ids in LDS (one-workgroup launch), or null: they were written by other workgroups.  VPL >= n_words.
template <int VPL, int GPW>
__device__ __forceinline__ void front_tail_few(const FrontArgs &a, SmallShared &sh, int n_pairs, const int32_t *ids_lds) {
    const int tid = threadIdx.x;
    const int wave = tid / MOE_WAVE, lane = tid % MOE_WAVE;
    const int E = a.E, n_inst = a.n_inst, C = a.C, p0 = wave * GPW * MOE_WAVE + lane;   // request g of this thread: p0 + g * MOE_WAVE
    int id[GPW];
#pragma unroll
    for (int g = 0; g < GPW; ++g) {
        const int p = p0 + g * MOE_WAVE;
        id[g] = -1;
        if (p < n_pairs) id[g] = ids_lds ? ids_lds[p] : __hip_atomic_load(a.ids + p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }

    // ---- Step 1; the slot of the request's expert here, or -1, and the request's place among its wavefront's for that slot
    int sl[GPW], rank[GPW];
#pragma unroll
    for (int g = 0; g < GPW; ++g) {
        sl[g] = -1;
        if (id[g] >= 0) {
            sh.sched.flag[id[g]] = 1u;
            sl[g] = sh.slot_of[id[g] * n_inst + a.g_self];
        }
    }
    int *run = &sh.perm.cnt[wave][0];                                 // this wavefront's requests of each slot so far
    const int slot_bits = C > 1 ? 32 - __builtin_clz(C - 1) : 1;
#pragma unroll
    for (int g = 0; g < GPW; ++g) {
        const uint64_t same = moe::lanes_alike(sl[g], slot_bits, __ballot(sl[g] >= 0));
        int before = 0;
        if (g > 0) {
            wave_lds_order();                                         // what the previous group's first lanes wrote
            if (sl[g] >= 0) before = run[sl[g]];
            wave_lds_order();                                         // every lane of a slot has read before its first lane writes
        }
        rank[g] = before + __popcll(same & moe::lanemask_lt());
        if (sl[g] >= 0 && lane == __builtin_ctzll(same)) run[sl[g]] = before + __popcll(same);
    }
    __syncthreads();

    // ---- Step 2 (first wavefront), slot_of in LDS; the prefix over the wavefronts meanwhile
    if (wave == 0) {
        const auto rep_of = [&](int e, int g) {
            const int single = sh.sched.single_rid[e], multi = (g < 0 ? 0 : g) * C + sh.slot_of[e * n_inst + (g < 0 ? 0 : g)];
            return g >= 0 ? multi : single;
        };
        const int load = moe::aebs_select_wave<VPL, VPL>(sh.sched.flag, sh.sched.host_mask, sh.sched.multi_mask,
                                                    sh.sched.single_mask, E, n_inst, a.n_words, lane, rep_of, sh.sched.rep,
                                                    a.act_rep);
        if (lane < n_inst) a.load[lane] = load;
    } else {
        for (int s = tid - MOE_WAVE; s < C; s += moe::kFrontThreads - MOE_WAVE) {
            int run = 0;
#pragma unroll
            for (int w = 0; w < moe::kFrontWaves; ++w) {
                const int c = sh.perm.cnt[w][s];
                sh.perm.cnt[w][s] = run;
                run += c;
            }
            sh.perm.total[s] = run;
        }
        for (int e = tid - MOE_WAVE; e < E; e += moe::kFrontThreads - MOE_WAVE) {
            const int s = sh.slot_of[e * n_inst + a.g_self];
            if (s >= 0) sh.expert_of[s] = static_cast<int16_t>(e);
        }
    }
    __syncthreads();

    // ---- Step 3; the second wavefront places the slots that Alg. 1 kept
    const int rid_lo = a.g_self * C;
    if (wave == 1) {
        const auto total_of = [&](int s) {
            static_assert((MOE_MAX_EXPERTS & (MOE_MAX_EXPERTS - 1)) == 0, "the mask keeps any value inside rep");
            const int e = sh.expert_of[s] & (MOE_MAX_EXPERTS - 1);    // unspecified for an empty slot, whose total is 0
            return sh.sched.rep[e] == rid_lo + s ? sh.perm.total[s] : 0;
        };
        static_assert(kFewPairs < 32768, "scan_slots_packed counts blocks in 16 bits");
        moe::scan_slots_packed(sh.perm, C, a.block_rows, total_of, a.slot_count, a.slot_off, lane);
    }
    int row[GPW];
#pragma unroll
    for (int g = 0; g < GPW; ++g) {
        row[g] = -1;
        if (id[g] >= 0) {
            const int r = sh.sched.rep[id[g]];
            a.rid[p0 + g * MOE_WAVE] = r;
            if (sl[g] >= 0 && r == rid_lo + sl[g]) row[g] = rank[g] + sh.perm.cnt[wave][sl[g]];
        }
    }
    __syncthreads();
    moe::list_blocks(sh.perm, C, a.block_rows, a.blocks);
#pragma unroll
    for (int g = 0; g < GPW; ++g) {
        if (id[g] >= 0) {
            const int p = p0 + g * MOE_WAVE;
            if (row[g] >= 0) {
                row[g] += sh.perm.off[sl[g]];
                a.perm[row[g]] = p;
            }
            a.pos[p] = row[g];
        }
    }
}

// What the last workgroup does.  A kernel for each, because the code of the tails that a batch does not run costs it scalar registers (256
// experts: 16 spilled in the selection, none here) and a longer way through the code.  All tails in one kernel and one each, us, this launch
// alone: E = 256, k = 8, T = 64 10.1 -> 9.7, T = 512 13.15 -> 12.9; E = 1000, k = 8, T = 700 24.4 -> 20.9; E = 64, k = 6, T = 1000 14.7 -> 14.5,
// T = 3000 19.2 -> 19.0; 101 sizes 0.86 to 1.01, median 0.98.
enum class Tail {
    Few,      // up to kFewPairs requests, layout table in LDS: front_tail_few
    Small,    // up to kRegPairs requests, layout table in LDS: front_tail_small
    Large,    // the others
};

template <int VPL, Tail TAIL>
__global__ __launch_bounds__(moe::kFrontThreads)
void front_kernel(FrontArgs a) {
    // the tails' LDS; the decode-size tail's is prepared while the tokens are routed, so the routing rows and
    // the ids have their own
    union Shared {
        moe::SchedShared sched;
        moe::PermShared perm;
        SmallShared small;
    };
    __shared__ Shared sh;
    __shared__ float row[moe::kFrontWaves][VPL * MOE_WAVE];
    __shared__ int32_t s_ids[TAIL == Tail::Few ? kSoloTokens * MOE_MAX_TOPK : 1];
    __shared__ int s_last;
    __shared__ uint32_t s_bits[kBitWords];                            // experts this workgroup's tokens selected

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / MOE_WAVE);
    const int lane = moe::lane_id();
    const int n_pairs = a.T * a.k;
    constexpr bool small = TAIL != Tail::Large;
    const bool solo = TAIL == Tail::Few && a.solo != 0;               // this is the only workgroup
    const bool bits = TAIL == Tail::Large && a.act_bits;
    TablePrefetch tp{};
    if (small) tp = prefetch_tables(a);
    if (bits) {
        if (threadIdx.x < kBitWords) s_bits[threadIdx.x] = 0u;
        __syncthreads();
    }
    // small batches route on a few wavefronts per workgroup (one or two per SIMD instead of four),
    // spread over more CUs: the selection is a long chain of cross-lane steps that four wavefronts
    // of one SIMD would take turns at
    for (int u = 0; u < a.tok_per_wave; ++u) {
        const int t = (blockIdx.x * a.tok_per_wave + u) * a.tok_per_wg + wave;
        if (wave < a.tok_per_wg && t < a.T) {
            const float *lg = a.logits + static_cast<size_t>(t) * a.E;
            int32_t *ids = a.ids + static_cast<size_t>(t) * a.k;
            float *w = a.w + static_cast<size_t>(t) * a.k;
            moe::route_token<VPL, true>(lg, a.E, a.k, a.cfg, row[wave], lane, ids, w, solo ? s_ids + t * a.k : nullptr,
                                        bits ? s_bits : nullptr);
        }
    }
    // Wavefronts that route nothing prepare the tail meanwhile, and so do those that have routed: against only the last workgroup preparing
    // it where all wavefronts route, E = 256, k = 4, T = 1025 12.7 -> 11.9 us, E = 128, k = 4, T = 1600 14.3 -> 14.05, E = 384, k = 2, T = 4000
    // 20.5 -> 20.3, none of 24 sizes slower.  Few requests are past 1024 tokens only with k = 1, and there the last workgroup does it: every
    // one would take 2 to 3 % off them, but without this test the code for all batches of few requests came out 0.5 to 2 % slower.
    const bool early = TAIL == Tail::Small || solo || a.tok_per_wg < moe::kFrontWaves;
    if (small && early) stage_small(a, sh.small, tp);
    if constexpr (TAIL == Tail::Few) {
        if (solo) {
            __syncthreads();
            front_tail_few<VPL, 1>(a, sh.small, n_pairs, s_ids);
            return;
        }
    }
    if (bits) {
        // Step 1 of Alg. 1, spread over the routing workgroups: one atomic per non-empty word
        __syncthreads();
        if (threadIdx.x < kBitWords && s_bits[threadIdx.x])
            __hip_atomic_fetch_or(a.act_bits + threadIdx.x, s_bits[threadIdx.x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // a workgroup barrier does not wait for global stores: the ticket must not overtake the ids
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
        const int old = __hip_atomic_fetch_add(a.ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s_last = old == static_cast<int>(gridDim.x) - 1;
        if (s_last) __hip_atomic_store(a.ticket, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // ready for the next call
    }
    __syncthreads();
    if (!s_last) return;

    if constexpr (small) {
        if (!early) {
            stage_small(a, sh.small, tp);
            __syncthreads();
        }
        if constexpr (TAIL == Tail::Few) {
            if (n_pairs <= kFewPairs / 2) front_tail_few<VPL, 1>(a, sh.small, n_pairs, nullptr);
            else front_tail_few<VPL, 2>(a, sh.small, n_pairs, nullptr);
        } else {
            if (n_pairs <= kRegPairs / 2) front_tail_small<VPL, kGpwMax / 2>(a, sh.small, n_pairs);
            else front_tail_small<VPL, kGpwMax>(a, sh.small, n_pairs);
        }
    } else {
        if (bits) {
            // Step 2 from the bitset the routing workgroups left; Step 3 and the sort follow in two launches
            moe::aebs_stage_tables(a.tb, sh.sched, a.E, a.n_inst, a.n_words);
            for (int e = threadIdx.x; e < a.E; e += moe::kFrontThreads) {
                const uint32_t word = __hip_atomic_load(a.act_bits + (e >> 5), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                sh.sched.flag[e] = (word >> (e & 31)) & 1u;
            }
            __syncthreads();
            if (threadIdx.x < kBitWords)                                  // ready for the next call
                __hip_atomic_store(a.act_bits + threadIdx.x, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            moe::aebs_select<VPL>(a.tb, sh.sched, a.E, a.n_inst, a.C, a.n_words, a.act_rep, a.load);
            return;
        }
        const int vec_ok = ((reinterpret_cast<uintptr_t>(a.ids) | reinterpret_cast<uintptr_t>(a.rid)) & 15) == 0;
        moe::aebs_block<VPL>(a.tb, sh.sched, a.E, a.n_inst, a.C, a.n_words, a.ids, n_pairs, vec_ok, true,
                        a.rid, a.act_rep, a.load);
        // rid is re-read below by other wavefronts of this workgroup
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        moe::permute_block(sh.perm, a.rid, n_pairs, a.g_self, a.C, a.slot_count, a.slot_off, a.perm, a.pos, a.blocks, a.block_rows);
    }
}

// Step 3 of Alg. 1 for one chunk of requests and the chunk's per-slot counts.
__global__ __launch_bounds__(moe::kFrontThreads)
void front_count_kernel(FrontArgs a) {
    __shared__ moe::PermShared sh;
    __shared__ int32_t rep[MOE_MAX_EXPERTS];
    for (int e = threadIdx.x; e < a.E; e += moe::kFrontThreads) rep[e] = a.act_rep[e];
    __syncthreads();
    const int n_pairs = a.T * a.k;
    const int p0 = blockIdx.x * a.chunk_pairs, p1 = min(n_pairs, p0 + a.chunk_pairs);
    moe::count_chunk(sh, rep, a.ids, a.rid, p0, p1, a.g_self, a.C, a.hist + blockIdx.x * a.C);
}

// The stable sort of one chunk into its places, from the counts of all chunks.
__global__ __launch_bounds__(moe::kFrontThreads)
void front_scatter_kernel(FrontArgs a) {
    __shared__ moe::PermShared sh;
    __shared__ int lower[MOE_MAX_SLOTS];
    const int n_pairs = a.T * a.k;
    const int p0 = blockIdx.x * a.chunk_pairs, p1 = min(n_pairs, p0 + a.chunk_pairs);
    moe::scatter_chunk(sh, lower, a.rid, p0, p1, blockIdx.x, a.n_chunks, a.hist, a.g_self, a.C, a.slot_count, a.slot_off,
                       a.perm, a.pos, a.blocks, a.block_rows);
}

constexpr int kFrontTwoTokens = 256 * moe::kFrontWaves;
template <int VPL>
int launch_front(const FrontArgs &a_in, const char *what, hipStream_t st) {
    FrontArgs a = a_in;
    // every routing workgroup takes a ticket from one counter: keep them to about a hundred
    const long long n_pairs = static_cast<long long>(a.T) * a.k;
    const Tail tail = n_pairs > kRegPairs || a.E * a.n_inst > kSlotOfLds ? Tail::Large : n_pairs > kFewPairs ? Tail::Small : Tail::Few;
    static_assert(kSoloTokens * MOE_MAX_TOPK <= kFewPairs, "a batch of one workgroup is one of few requests");
    a.solo = tail == Tail::Few && a.T <= solo_tokens(a.E, a.k);
    a.tok_per_wg = a.solo ? moe::kFrontWaves : a.T <= 512 ? 4 : a.T <= 1024 ? 8 : moe::kFrontWaves;
    // past one workgroup per CU the counter and the bit set cost more than a second token on every wavefront
    // (T = 8192, k = 8, this launch and the two behind it: E = 256 30.6 -> 26.2 us; E = 128 31.8 -> 27.6)
    a.tok_per_wave = a.act_bits && a.T > kFrontTwoTokens ? 2 : 1;
    const int per = a.tok_per_wg * a.tok_per_wave;
    const int blocks = a.T > 0 ? (a.T + per - 1) / per : 1;
    const dim3 grid(blocks), threads(moe::kFrontThreads);
    if (tail == Tail::Few) hipLaunchKernelGGL((front_kernel<VPL, Tail::Few>), grid, threads, 0, st, a);
    else if (tail == Tail::Small) hipLaunchKernelGGL((front_kernel<VPL, Tail::Small>), grid, threads, 0, st, a);
    else hipLaunchKernelGGL((front_kernel<VPL, Tail::Large>), grid, threads, 0, st, a);
    if (a.act_bits) {
        hipLaunchKernelGGL(front_count_kernel, dim3(a.n_chunks), dim3(moe::kFrontThreads), 0, st, a);
        hipLaunchKernelGGL(front_scatter_kernel, dim3(a.n_chunks), dim3(moe::kFrontThreads), 0, st, a);
    }
    return moe::check_launch(what);
}

// Batches whose requests do not fit the registers of one workgroup (or whose layout table does not
// fit its LDS) take the chunked tail.
bool front_is_large(const moe_placement_t *pl, int T, int k) {
    return static_cast<long long>(T) * k > kRegPairs || pl->E * pl->n_inst > kSlotOfLds;
}

int launch_front_for(const FrontArgs &a, const char *what, hipStream_t st) {
    const int vpl = (a.E + MOE_WAVE - 1) / MOE_WAVE;
    if (vpl <= 1) return launch_front<1>(a, what, st);
    if (vpl <= 2) return launch_front<2>(a, what, st);
    if (vpl <= 4) return launch_front<4>(a, what, st);
    if (vpl <= 8) return launch_front<8>(a, what, st);
    if (vpl <= 12) return launch_front<12>(a, what, st);      // E = 640, k = 16, T = 55: 14.7 us, 17.2 with the code for 1024 experts
    return launch_front<16>(a, what, st);
}

int check_selection(int T, int E, int k, const moe_route_cfg *cfg) {
    if (!cfg || T < 0 || E < 1 || k < 1 || k > E) return MOE_EINVAL;
    if (E > MOE_MAX_EXPERTS || k > MOE_MAX_TOPK) return MOE_ESHAPE;
    if (static_cast<long long>(T) * k > 0x7fffffffLL) return MOE_ESHAPE;
    if (cfg->mode != MOE_ROUTE_SOFTMAX && cfg->mode != MOE_ROUTE_SIGMOID_GROUP) return MOE_EINVAL;
    if (cfg->mode == MOE_ROUTE_SIGMOID_GROUP) {
        if (cfg->n_group < 1 || cfg->topk_group < 1 || cfg->topk_group > cfg->n_group) return MOE_EINVAL;
        if (cfg->n_group > 64 || E % cfg->n_group != 0 || E / cfg->n_group < 2) return MOE_ESHAPE;
        if (k > cfg->topk_group * (E / cfg->n_group)) return MOE_EINVAL;
    }
    return MOE_OK;
}

// the gate's operands: bf16 rows of d_h elements read 16 bytes at a time
int check_gate(const void *X, const void *Wr, const float *bias, const float *logits, int T, int E, int d_h) {
    if (d_h < 32 || d_h % 32 != 0) return MOE_ESHAPE;
    if (static_cast<long long>(T) * E > 0x7fffffffLL) return MOE_ESHAPE;
    if (!Wr || !moe::aligned(Wr, 16) || !moe::aligned(bias, 4)) return MOE_EINVAL;
    if (T > 0 && (!X || !logits || !moe::aligned(X, 16) || !moe::aligned(logits, 4))) return MOE_EINVAL;
    return MOE_OK;
}

int fill_tail(FrontArgs &a, const moe_placement_t *pl, int g_self, int T, int32_t *rid_dev, int32_t *act_rep_dev,
              int32_t *load_dev, int32_t *slot_count_dev, int32_t *slot_off_dev, int32_t *perm_dev, int32_t *pos_dev,
              int32_t *blocks_dev) {
    if (g_self < 0 || g_self >= pl->n_inst) return MOE_EINVAL;
    if (!act_rep_dev || !load_dev || !slot_count_dev || !slot_off_dev || !blocks_dev) return MOE_EINVAL;
    if (T > 0 && (!rid_dev || !perm_dev || !pos_dev)) return MOE_EINVAL;
    const void *ptrs[] = {rid_dev, act_rep_dev, load_dev, slot_count_dev, slot_off_dev, perm_dev, pos_dev};
    for (const void *p : ptrs)
        if (!moe::aligned(p, 4)) return MOE_EINVAL;
    if (!moe::aligned(blocks_dev, 16)) return MOE_EINVAL;
    a.tb = moe::SchedTables{pl->host_mask_d, pl->slot_of_d, pl->single_rid_d, pl->multi_mask_d, pl->single_mask_d};
    a.n_inst = pl->n_inst; a.C = pl->C; a.n_words = pl->n_words; a.g_self = g_self;
    a.rid = rid_dev; a.act_rep = act_rep_dev; a.load = load_dev;
    a.slot_count = slot_count_dev; a.slot_off = slot_off_dev; a.perm = perm_dev; a.pos = pos_dev; a.blocks = blocks_dev;
    a.block_rows = moe::ffn_block_rows(T);
    return MOE_OK;
}

}  // namespace

extern "C" int moe_route_schedule_permute(const moe_placement_t *pl, int g_self, const float *logits_dev, int T, int k,
                                          const moe_route_cfg *cfg, int32_t *topk_ids_dev, float *topk_w_dev,
                                          int32_t *rid_dev, int32_t *act_rep_dev, int32_t *load_dev,
                                          int32_t *slot_count_dev, int32_t *slot_off_dev, int32_t *perm_dev,
                                          int32_t *pos_dev, int32_t *blocks_dev, int32_t *sync_dev, void *stream) {
    if (!pl) return MOE_EINVAL;
    const int E = pl->E;
    if (const int rc = check_selection(T, E, k, cfg)) return rc;
    if (!sync_dev || !moe::aligned(sync_dev, 4)) return MOE_EINVAL;
    if (T > 0 && (!logits_dev || !topk_ids_dev || !topk_w_dev)) return MOE_EINVAL;
    if (!moe::aligned(logits_dev, 4) || !moe::aligned(topk_ids_dev, 4) || !moe::aligned(topk_w_dev, 4)) return MOE_EINVAL;
    FrontArgs a{};
    if (const int rc = fill_tail(a, pl, g_self, T, rid_dev, act_rep_dev, load_dev, slot_count_dev, slot_off_dev,
                                 perm_dev, pos_dev, blocks_dev))
        return rc;
    a.logits = logits_dev; a.T = T; a.E = E; a.k = k; a.cfg = *cfg;
    a.ids = topk_ids_dev; a.w = topk_w_dev;
    a.ticket = sync_dev;
    if (T > 0 && front_is_large(pl, T, k)) {
        a.act_bits = reinterpret_cast<uint32_t *>(sync_dev + 1);
        a.hist = sync_dev + 1 + kBitWords;
        a.chunk_pairs = kChunkPairs;
        a.n_chunks = static_cast<int>((static_cast<long long>(T) * k + kChunkPairs - 1) / kChunkPairs);
    }
    return launch_front_for(a, "moe_route_schedule_permute", static_cast<hipStream_t>(stream));
}

extern "C" size_t moe_front_sync_len(const moe_placement_t *pl, int T, int k) {
    if (!pl || T < 0 || k < 1) return 0;
    if (T == 0 || !front_is_large(pl, T, k)) return 1;
    const size_t n_chunks = (static_cast<size_t>(T) * k + kChunkPairs - 1) / kChunkPairs;
    return 1 + kBitWords + n_chunks * pl->C;
}

extern "C" size_t moe_gate_sync_len(int T) { return T > 0 ? 1 + (static_cast<size_t>(T) + 15) / 16 : 1; }

extern "C" int moe_gate_route(const void *X_dev, const void *Wr_dev, const float *bias_dev, int T, int E, int d_h, int k,
                              const moe_route_cfg *cfg, float *logits_dev, int32_t *topk_ids_dev, float *topk_w_dev,
                              int32_t *sync_dev, void *stream) {
    if (const int rc = check_selection(T, E, k, cfg)) return rc;
    if (const int rc = check_gate(X_dev, Wr_dev, bias_dev, logits_dev, T, E, d_h)) return rc;
    if (!sync_dev || !moe::aligned(sync_dev, 4)) return MOE_EINVAL;
    if (T == 0) return MOE_OK;
    if (!topk_ids_dev || !topk_w_dev || !moe::aligned(topk_ids_dev, 4) || !moe::aligned(topk_w_dev, 4)) return MOE_EINVAL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (const int rc = launch_gate(X_dev, Wr_dev, bias_dev, logits_dev, T, E, d_h, st)) return rc;
    return moe_route(logits_dev, T, E, k, cfg, topk_ids_dev, topk_w_dev, stream);
}

extern "C" int moe_gate_route_schedule_permute(const moe_placement_t *pl, int g_self, const void *X_dev,
                                               const void *Wr_dev, const float *bias_dev, int T, int d_h, int k,
                                               const moe_route_cfg *cfg, float *logits_dev, int32_t *topk_ids_dev,
                                               float *topk_w_dev, int32_t *rid_dev, int32_t *act_rep_dev,
                                               int32_t *load_dev, int32_t *slot_count_dev, int32_t *slot_off_dev,
                                               int32_t *perm_dev, int32_t *pos_dev, int32_t *blocks_dev,
                                               int32_t *sync_dev, void *stream) {
    if (!pl) return MOE_EINVAL;
    const int E = pl->E;
    if (const int rc = check_selection(T, E, k, cfg)) return rc;
    if (const int rc = check_gate(X_dev, Wr_dev, bias_dev, logits_dev, T, E, d_h)) return rc;
    if (!sync_dev || !moe::aligned(sync_dev, 4)) return MOE_EINVAL;
    if (T > 0 && (!topk_ids_dev || !topk_w_dev)) return MOE_EINVAL;
    if (!moe::aligned(topk_ids_dev, 4) || !moe::aligned(topk_w_dev, 4)) return MOE_EINVAL;
    FrontArgs a{};
    if (const int rc = fill_tail(a, pl, g_self, T, rid_dev, act_rep_dev, load_dev, slot_count_dev, slot_off_dev,
                                 perm_dev, pos_dev, blocks_dev))
        return rc;
    a.T = T; a.E = E; a.k = k; a.cfg = *cfg;
    a.logits = logits_dev;
    a.ids = topk_ids_dev; a.w = topk_w_dev;
    a.ticket = sync_dev;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (T > 0)
        if (const int rc = launch_gate(X_dev, Wr_dev, bias_dev, logits_dev, T, E, d_h, st)) return rc;
    return launch_front_for(a, "moe_gate_route_schedule_permute", st);
}
