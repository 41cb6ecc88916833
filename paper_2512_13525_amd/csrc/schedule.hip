// a1-a3: Activated-Expert-Balanced Scheduling (Janus Sec. 3.4, Alg. 1) as one kernel of one
// workgroup; the algorithm itself lives in dispatch_dev.h (aebs_block).
#include "dispatch_dev.h"

namespace {

using moe::SchedTables;
constexpr int kSchedThreads = moe::kFrontThreads;

// One workgroup per batch (blockIdx.x): batch b reads ids + b*n_pairs and writes rid + b*n_pairs,
// act_rep + b*E, load_out + b*n_inst.  The single-batch call is a grid of one.
// W: 64-expert words the selection is compiled for (n_words <= W); G: words it reads at once.
template <int W, int G>
__global__ __launch_bounds__(kSchedThreads, G <= 4 ? 8 : 4)           // 8 wavefronts a SIMD: two workgroups a CU
void aebs_kernel(SchedTables tb, int E, int n_inst, int C, int n_words,
                 const int32_t *__restrict__ ids, int n_pairs, int vec_ok,
                 int32_t *__restrict__ rid, int32_t *__restrict__ act_rep, int32_t *__restrict__ load_out) {
    __shared__ moe::SchedShared sh;
    const size_t b = blockIdx.x;
    moe::aebs_block<W, G>(tb, sh, E, n_inst, C, n_words, ids + b * n_pairs, n_pairs, vec_ok, false,
                    rid ? rid + b * n_pairs : nullptr, act_rep ? act_rep + b * E : nullptr, load_out + b * n_inst);
}

// Loads only, many batches: one wavefront per batch, no barrier, no rewriting.  The four wavefronts of a workgroup
// share the layout tables and walk the batches with a stride of the whole grid.  A batch is one pass over its ids
// (16-byte loads, eight in flight a lane, whatever the batch's own alignment), flags in wave-private LDS, then the same selection as aebs_kernel.
constexpr int kLoadsWaves = 4;
template <int W>
__global__ __launch_bounds__(kLoadsWaves * MOE_WAVE)
void aebs_loads_kernel(SchedTables tb, int E, int n_inst, int n_words, const int32_t *__restrict__ ids, int n_batches,
                       int n_pairs, int32_t *__restrict__ load_out) {
    __shared__ uint64_t host_mask[W * MOE_WAVE], multi_mask[W], single_mask[MOE_MAX_INSTANCES * W];
    __shared__ uint32_t flags[kLoadsWaves][W * MOE_WAVE];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / MOE_WAVE), lane = moe::lane_id();
    uint32_t *flag = flags[wave];
    for (int e = threadIdx.x; e < E; e += kLoadsWaves * MOE_WAVE) host_mask[e] = tb.host_mask[e];
    if (threadIdx.x < n_words) multi_mask[threadIdx.x] = tb.multi_mask[threadIdx.x];
    for (int i = threadIdx.x; i < n_inst * n_words; i += kLoadsWaves * MOE_WAVE) single_mask[i] = tb.single_mask[i];
    __syncthreads();
    constexpr int kAhead = 8;
    for (int b = blockIdx.x * kLoadsWaves + wave; b < n_batches; b += gridDim.x * kLoadsWaves) {
        const int32_t *my = ids + static_cast<size_t>(b) * n_pairs;
#pragma unroll
        for (int w = 0; w < W; ++w) flag[w * MOE_WAVE + lane] = 0u;
        __builtin_amdgcn_wave_barrier();                             // LDS operations of a wavefront stay in order
        // whole 16 bytes from the first aligned one on; up to three ids before them and after them
        const int lead = static_cast<int>(-(reinterpret_cast<uintptr_t>(my) >> 2) & 3);
        const int head = lead < n_pairs ? lead : n_pairs, n4 = (n_pairs - head) >> 2, tail = head + (n4 << 2);
        if (lane < head) flag[my[lane]] = 1u;
        if (lane < n_pairs - tail) flag[my[tail + lane]] = 1u;
        const int4 *my4 = reinterpret_cast<const int4 *>(my + head);
        for (int i0 = 0; i0 < n4; i0 += kAhead * MOE_WAVE) {
            int4 v[kAhead];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const int i = i0 + u * MOE_WAVE + lane;
                v[u] = my4[i < n4 ? i : n4 - 1];                     // past the end: the last four again
            }
#pragma unroll
            for (int u = 0; u < kAhead; ++u) { flag[v[u].x] = 1u; flag[v[u].y] = 1u; flag[v[u].z] = 1u; flag[v[u].w] = 1u; }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const auto no_rep = [](int, int) { return -1; };
        const int load = moe::aebs_select_wave<W, W < 4 ? W : 4>(flag, host_mask, multi_mask, single_mask, E, n_inst, n_words, lane,
                                                  no_rep, static_cast<int32_t *>(nullptr), static_cast<int32_t *>(nullptr));
        if (lane < n_inst) load_out[static_cast<size_t>(b) * n_inst + lane] = load;
        __builtin_amdgcn_wave_barrier();
    }
}

// Baseline policies the paper compares AEBS with (Sec. 5): every request of expert e goes to e's
// first replica (MOE_POLICY_HOME: no scheduling), or to replica number draw mod R(e) of e, replicas
// in ascending instance order (MOE_POLICY_RANDOM: balances tokens, not activated experts).  One
// workgroup; load[g] = distinct replicas of instance g that received a request, counted through a
// bitset of all n_inst*C replica ids in LDS.
__global__ __launch_bounds__(kSchedThreads)
void baseline_kernel(const uint64_t *__restrict__ host_mask, const int16_t *__restrict__ slot_of, int n_inst, int C,
                     const int32_t *__restrict__ ids, const uint32_t *__restrict__ draws, int n_pairs, int policy,
                     int32_t *__restrict__ rid, int32_t *__restrict__ load_out) {
    __shared__ uint32_t used[MOE_MAX_INSTANCES * MOE_MAX_SLOTS / 32];
    __shared__ int load[MOE_MAX_INSTANCES];
    const int n_rids = n_inst * C;
    // one workgroup per batch
    ids += static_cast<size_t>(blockIdx.x) * n_pairs;
    if (draws) draws += static_cast<size_t>(blockIdx.x) * n_pairs;
    if (rid) rid += static_cast<size_t>(blockIdx.x) * n_pairs;
    load_out += static_cast<size_t>(blockIdx.x) * n_inst;
    for (int i = threadIdx.x; i < (n_rids + 31) / 32; i += kSchedThreads) used[i] = 0u;
    if (threadIdx.x < n_inst) load[threadIdx.x] = 0;
    __syncthreads();
    for (int p = threadIdx.x; p < n_pairs; p += kSchedThreads) {
        const int e = ids[p];
        uint64_t hosts = host_mask[e];
        int skip = policy == MOE_POLICY_RANDOM ? static_cast<int>(draws[p] % static_cast<uint32_t>(__popcll(hosts))) : 0;
        while (skip-- > 0) hosts &= hosts - 1;                   // drop the lowest instances
        const int g = __builtin_ctzll(hosts);
        const int r = g * C + slot_of[e * n_inst + g];
        if (rid) rid[p] = r;
        atomicOr(&used[r >> 5], 1u << (r & 31));
    }
    __syncthreads();
    for (int r = threadIdx.x; r < n_rids; r += kSchedThreads)
        if ((used[r >> 5] >> (r & 31)) & 1u) atomicAdd(&load[r / C], 1);
    __syncthreads();
    if (threadIdx.x < n_inst) load_out[threadIdx.x] = load[threadIdx.x];
}

void launch_aebs(const moe_placement_t *pl, int n_batches, const int32_t *ids, int n_pairs, int vec_ok, int32_t *rid,
                 int32_t *act_rep, int32_t *load, hipStream_t st) {
    const SchedTables tb{pl->host_mask_d, pl->slot_of_d, pl->single_rid_d, pl->multi_mask_d, pl->single_mask_d};
#define MOE_AEBS(W, G) hipLaunchKernelGGL((aebs_kernel<W, G>), dim3(n_batches), dim3(kSchedThreads), 0, st, tb, pl->E, pl->n_inst, \
                                          pl->C, pl->n_words, ids, n_pairs, vec_ok, rid, act_rep, load)
    // more than four words: all at once takes a workgroup 68 to 128 registers, so only where one workgroup has a CU to itself
    // (E = 312, k = 4, one batch of 11 tokens: 3.8 us, 4.5 in groups of four; E = 1024, 512 batches: 11.6 and 8.6)
    if (pl->n_words <= 1) MOE_AEBS(1, 1);
    else if (pl->n_words <= 2) MOE_AEBS(2, 2);
    else if (pl->n_words <= 4) MOE_AEBS(4, 4);
    else if (n_batches > 256) MOE_AEBS(16, 4);
    else if (pl->n_words <= 8) MOE_AEBS(8, 8);
    else MOE_AEBS(16, 16);
#undef MOE_AEBS
}

// A workgroup per batch keeps two batches on each CU, 512 in all; from the second round on a wavefront per batch
// is faster as long as its pass over the ids (2048 at a time, one such step after the other) is short against the rounds
// it replaces (2000 batches of 2048 requests 4.7 us a call against 9.8, 5000 of 8192 28 against 37, 600 of 4096 4.7 against
// 5.8; but 513 of 8192 6.6 against 6.1, 2000 of 32768 44 against 40).
bool loads_by_wavefront(int n_batches, int n_pairs) { return n_batches > 512 && n_pairs <= 8192 && n_pairs / 8 <= n_batches; }
void launch_loads(const moe_placement_t *pl, int n_batches, const int32_t *ids, int n_pairs, int32_t *load, hipStream_t st) {
    const SchedTables tb{pl->host_mask_d, pl->slot_of_d, pl->single_rid_d, pl->multi_mask_d, pl->single_mask_d};
    const long long wanted = (static_cast<long long>(n_batches) + kLoadsWaves - 1) / kLoadsWaves;
    const unsigned grid = static_cast<unsigned>(wanted < 2048 ? wanted : 2048);
#define MOE_LOADS(W) hipLaunchKernelGGL(aebs_loads_kernel<W>, dim3(grid), dim3(kLoadsWaves * MOE_WAVE), 0, st, tb, pl->E, pl->n_inst, \
                                        pl->n_words, ids, n_batches, n_pairs, load)
    if (pl->n_words <= 1) MOE_LOADS(1);
    else if (pl->n_words <= 2) MOE_LOADS(2);
    else if (pl->n_words <= 4) MOE_LOADS(4);
    else if (pl->n_words <= 8) MOE_LOADS(8);
    else MOE_LOADS(16);
#undef MOE_LOADS
}

}  // namespace

extern "C" int moe_schedule_baseline(const moe_placement_t *pl, const int32_t *topk_ids_dev, int T, int k,
                                     int policy, const uint32_t *draws_dev, int32_t *rid_dev, int32_t *load_dev,
                                     void *stream) {
    if (!pl || T < 0 || k < 1) return MOE_EINVAL;
    if (policy != MOE_POLICY_HOME && policy != MOE_POLICY_RANDOM) return MOE_EINVAL;
    if (k > MOE_MAX_TOPK) return MOE_ESHAPE;
    if (static_cast<long long>(T) * k > 0x7fffffffLL) return MOE_ESHAPE;
    if (!load_dev) return MOE_EINVAL;
    if (T > 0 && (!topk_ids_dev || !rid_dev || (policy == MOE_POLICY_RANDOM && !draws_dev))) return MOE_EINVAL;
    if (!moe::aligned(topk_ids_dev, 4) || !moe::aligned(rid_dev, 4) || !moe::aligned(draws_dev, 4) ||
        !moe::aligned(load_dev, 4))
        return MOE_EINVAL;
    hipLaunchKernelGGL(baseline_kernel, dim3(1), dim3(kSchedThreads), 0, static_cast<hipStream_t>(stream),
                       pl->host_mask_d, pl->slot_of_d, pl->n_inst, pl->C, topk_ids_dev, draws_dev, T * k, policy,
                       rid_dev, load_dev);
    return moe::check_launch("moe_schedule_baseline");
}

extern "C" int moe_schedule(const moe_placement_t *pl, const int32_t *topk_ids_dev, int T, int k,
                            int32_t *rid_dev, int32_t *act_rep_dev, int32_t *load_dev, void *stream) {
    if (!pl || T < 0 || k < 1) return MOE_EINVAL;
    if (k > MOE_MAX_TOPK) return MOE_ESHAPE;
    if (static_cast<long long>(T) * k > 0x7fffffffLL) return MOE_ESHAPE;
    if (!act_rep_dev || !load_dev) return MOE_EINVAL;
    if (T > 0 && (!topk_ids_dev || !rid_dev)) return MOE_EINVAL;
    if (!moe::aligned(topk_ids_dev, 4) || !moe::aligned(rid_dev, 4) || !moe::aligned(act_rep_dev, 4) ||
        !moe::aligned(load_dev, 4))
        return MOE_EINVAL;
    const int vec_ok = moe::aligned(topk_ids_dev, 16) && moe::aligned(rid_dev, 16);
    launch_aebs(pl, 1, topk_ids_dev, T * k, vec_ok, rid_dev, act_rep_dev, load_dev, static_cast<hipStream_t>(stream));
    return moe::check_launch("moe_schedule");
}

// The batched forms for the Monte-Carlo estimate of a_max(n_e, B) (Sec. 3.5: the table Alg. 2 reads is built
// by sampling batches and scheduling them): one launch, one workgroup per sampled batch.
extern "C" int moe_schedule_batched(const moe_placement_t *pl, const int32_t *topk_ids_dev, int n_batches, int T, int k,
                                    int32_t *rid_dev, int32_t *act_rep_dev, int32_t *load_dev, void *stream) {
    if (!pl || n_batches < 0 || T < 0 || k < 1) return MOE_EINVAL;
    if (k > MOE_MAX_TOPK) return MOE_ESHAPE;
    if (static_cast<long long>(T) * k > 0x7fffffffLL || n_batches > 0x7fffffff / 2) return MOE_ESHAPE;
    if (n_batches == 0) return MOE_OK;
    if (!load_dev || (T > 0 && !topk_ids_dev)) return MOE_EINVAL;
    if (!moe::aligned(topk_ids_dev, 4) || !moe::aligned(rid_dev, 4) || !moe::aligned(act_rep_dev, 4) ||
        !moe::aligned(load_dev, 4))
        return MOE_EINVAL;
    // 16-byte accesses need every batch's rows aligned, not only the first
    const int vec_ok = moe::aligned(topk_ids_dev, 16) && (!rid_dev || moe::aligned(rid_dev, 16)) &&
                       (static_cast<long long>(T) * k) % 4 == 0;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (!rid_dev && !act_rep_dev && loads_by_wavefront(n_batches, T * k))
        launch_loads(pl, n_batches, topk_ids_dev, T * k, load_dev, st);
    else
        launch_aebs(pl, n_batches, topk_ids_dev, T * k, vec_ok, rid_dev, act_rep_dev, load_dev, st);
    return moe::check_launch("moe_schedule_batched");
}

extern "C" int moe_schedule_baseline_batched(const moe_placement_t *pl, const int32_t *topk_ids_dev, int n_batches, int T,
                                             int k, int policy, const uint32_t *draws_dev, int32_t *rid_dev,
                                             int32_t *load_dev, void *stream) {
    if (!pl || n_batches < 0 || T < 0 || k < 1) return MOE_EINVAL;
    if (policy != MOE_POLICY_HOME && policy != MOE_POLICY_RANDOM) return MOE_EINVAL;
    if (k > MOE_MAX_TOPK) return MOE_ESHAPE;
    if (static_cast<long long>(T) * k > 0x7fffffffLL || n_batches > 0x7fffffff / 2) return MOE_ESHAPE;
    if (n_batches == 0) return MOE_OK;
    if (!load_dev) return MOE_EINVAL;
    if (T > 0 && (!topk_ids_dev || (policy == MOE_POLICY_RANDOM && !draws_dev))) return MOE_EINVAL;
    if (!moe::aligned(topk_ids_dev, 4) || !moe::aligned(rid_dev, 4) || !moe::aligned(draws_dev, 4) ||
        !moe::aligned(load_dev, 4))
        return MOE_EINVAL;
    hipLaunchKernelGGL(baseline_kernel, dim3(n_batches), dim3(kSchedThreads), 0, static_cast<hipStream_t>(stream),
                       pl->host_mask_d, pl->slot_of_d, pl->n_inst, pl->C, topk_ids_dev,
                       policy == MOE_POLICY_RANDOM ? draws_dev : nullptr, T * k, policy, rid_dev, load_dev);
    return moe::check_launch("moe_schedule_baseline_batched");
}
