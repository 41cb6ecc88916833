// a4: this instance's share of the dispatch (Janus Sec. 3.4, Step 4) and
// a6: the weighted top-k combine that produces the instance-partial output entering the
// reverse-path reduction (Sec. 3.3).  The counting sort lives in dispatch_dev.h (permute_block).
#include "dispatch_dev.h"

namespace {

constexpr int kPermThreads = moe::kFrontThreads;

__global__ __launch_bounds__(kPermThreads)
void permute_kernel(const int32_t *__restrict__ rid, int n_pairs, int g_self, int C,
                    int32_t *__restrict__ slot_count, int32_t *__restrict__ slot_off,
                    int32_t *__restrict__ perm, int32_t *__restrict__ pos, int32_t *__restrict__ blocks,
                    int block_rows) {
    __shared__ moe::PermShared sh;
    moe::permute_block(sh, rid, n_pairs, g_self, C, slot_count, slot_off, perm, pos, blocks, block_rows);
}

// The dispatch of a shared expert: one slot that every token visits once (identity permutation),
// cut into the same blocks of rows as any other slot.
__global__ __launch_bounds__(256)
void shared_dispatch_kernel(int T, int block_rows, int32_t *__restrict__ slot_off, int32_t *__restrict__ perm,
                            int32_t *__restrict__ blocks) {
    const int tid = blockIdx.x * blockDim.x + threadIdx.x, n = gridDim.x * blockDim.x;
    const int n_blocks = (T + block_rows - 1) / block_rows;
    if (tid == 0) {
        slot_off[0] = 0;
        slot_off[1] = T;
        reinterpret_cast<int4 *>(blocks)[0] = make_int4(n_blocks, block_rows, T > 64 ? (T + 63) / 64 : 0, T > 64 ? (T + 127) / 128 : 0);
    }
    for (int i = tid; i < T; i += n) perm[i] = i;
    for (int b = tid; b < n_blocks; b += n) reinterpret_cast<int4 *>(blocks)[1 + b] = make_int4(0, b * block_rows, T, 0);
}

// One workgroup per (token, chunk of 256*V columns); each thread owns V consecutive columns (V = 8: one 16-byte store of
// bf16; V = 4 where the columns or the output's alignment ask for it).  Bound by memory: the output once, the local rows of Yp once.
// The token's k places and weights are read by the first lanes of every wavefront at once and handed round with lane
// reads, so a token without a local request stores its zeros after one load, and the rows of one with several follow
// each other without a load of pos in between (two in flight).  T = 8192, d_h = 4096, k = 8: 22 us against 34 with a loop
// over k that reads pos[j] before every row.
// Ys (optional): rows of a shared expert's output, added with weight 1 after the routed sum.
template <bool OUT_BF16, int V>
__global__ __launch_bounds__(256)
void combine_kernel(const float *__restrict__ Yp, const int32_t *__restrict__ pos,
                    const float *__restrict__ w, const float *__restrict__ Ys, int k, int d_h, void *__restrict__ Y) {
    constexpr int N = V / 4;
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    const int i = blockIdx.x;
    if ((blockIdx.y * 256 + (threadIdx.x & ~(MOE_WAVE - 1))) * V >= static_cast<unsigned>(d_h)) return;   // wavefronts past the columns
    const int col0 = (blockIdx.y * 256 + threadIdx.x) * V;
    const bool on = col0 < d_h;                                       // threads past the columns stay for the lane reads
    const int col = on ? col0 : 0;
    const int lane = moe::lane_id();
    int r_l = -1;
    float w_l = 0.f;
    if (lane < k) {                                                   // k <= 32
        r_l = pos[static_cast<size_t>(i) * k + lane];
        w_l = w[static_cast<size_t>(i) * k + lane];
    }
    uint64_t todo = __ballot(r_l >= 0);
    f32x4 acc[N];
#pragma unroll
    for (int n = 0; n < N; ++n) acc[n] = f32x4{0.f, 0.f, 0.f, 0.f};
    const auto row = [&](int j, f32x4 (&y)[N]) {
        const float *p = Yp + static_cast<size_t>(__builtin_amdgcn_readlane(r_l, j)) * d_h + col;
#pragma unroll
        for (int n = 0; n < N; ++n) y[n] = *reinterpret_cast<const f32x4 *>(p + 4 * n);
    };
    const auto add = [&](int j, const f32x4 (&y)[N]) {
        const float wj = __uint_as_float(static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(__float_as_uint(w_l)), j)));
#pragma unroll
        for (int n = 0; n < N; ++n)
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[n][q] += wj * y[n][q];
    };
    while (todo) {                                                    // ascending j
        const int j0 = __builtin_ctzll(todo);
        todo &= todo - 1;
        f32x4 y0[N], y1[N];
        row(j0, y0);
        if (todo) {
            const int j1 = __builtin_ctzll(todo);
            todo &= todo - 1;
            row(j1, y1);
            add(j0, y0);
            add(j1, y1);
        } else {
            add(j0, y0);
        }
    }
    if (Ys) {
        const float *p = Ys + static_cast<size_t>(i) * d_h + col;
#pragma unroll
        for (int n = 0; n < N; ++n) acc[n] += *reinterpret_cast<const f32x4 *>(p + 4 * n);
    }
    if (!on) return;
    if (OUT_BF16) {
        typedef uint16_t u16xV __attribute__((ext_vector_type(V)));
        u16xV o;
#pragma unroll
        for (int n = 0; n < N; ++n)
#pragma unroll
            for (int q = 0; q < 4; ++q) o[n * 4 + q] = moe::f32_to_bf16(acc[n][q]);
        *reinterpret_cast<u16xV *>(static_cast<uint16_t *>(Y) + static_cast<size_t>(i) * d_h + col) = o;
    } else {
#pragma unroll
        for (int n = 0; n < N; ++n)
            *reinterpret_cast<f32x4 *>(static_cast<float *>(Y) + static_cast<size_t>(i) * d_h + col + 4 * n) = acc[n];
    }
}

}  // namespace

extern "C" int moe_permute(const moe_placement_t *pl, int g_self, const int32_t *rid_dev, int T, int k,
                           int32_t *slot_count_dev, int32_t *slot_off_dev, int32_t *perm_dev,
                           int32_t *pos_dev, int32_t *blocks_dev, void *stream) {
    if (!pl || T < 0 || k < 1) return MOE_EINVAL;
    if (g_self < 0 || g_self >= pl->n_inst) return MOE_EINVAL;
    if (k > MOE_MAX_TOPK) return MOE_ESHAPE;
    if (static_cast<long long>(T) * k > 0x7fffffffLL) return MOE_ESHAPE;
    if (!slot_count_dev || !slot_off_dev || !blocks_dev) return MOE_EINVAL;
    if (T > 0 && (!rid_dev || !perm_dev || !pos_dev)) return MOE_EINVAL;
    if (!moe::aligned(rid_dev, 4) || !moe::aligned(slot_count_dev, 4) || !moe::aligned(slot_off_dev, 4) ||
        !moe::aligned(perm_dev, 4) || !moe::aligned(pos_dev, 4) || !moe::aligned(blocks_dev, 16))
        return MOE_EINVAL;
    hipLaunchKernelGGL(permute_kernel, dim3(1), dim3(kPermThreads), 0, static_cast<hipStream_t>(stream),
                       rid_dev, T * k, g_self, pl->C, slot_count_dev, slot_off_dev, perm_dev, pos_dev, blocks_dev,
                       moe::ffn_block_rows(T));
    return moe::check_launch("moe_permute");
}

extern "C" size_t moe_max_blocks(int T, int k, int C) {
    if (T < 0 || k < 1 || C < 1) return 0;
    return static_cast<size_t>(moe::ffn_max_blocks(T, k, C));
}

extern "C" int moe_block_rows(int T) { return T < 0 ? 0 : moe::ffn_block_rows(T); }

extern "C" size_t moe_block_list_len(int T, int k, int C) {
    if (T < 0 || k < 1 || C < 1) return 0;
    return 4 * (1 + static_cast<size_t>(moe::ffn_max_blocks(T, k, C)));
}

namespace {

// Eight columns a thread from this many outputs on (T = 8192, d_h = 4096: 22 us with eight, 27 with four; level at T = 512,
// d_h = 7168; 6 to 16 % faster with 5 to 12 % of the requests local, 1 to 6 % slower with 30 to 60 %), where a row fills a
// wavefront of them (T = 33000, d_h = 128, 60 % local: 42 us with eight columns and all wavefronts kept, 20 so).
constexpr long long kCombineWide = 4 << 20;
constexpr int kCombineWideMinCols = MOE_WAVE * 8;

int combine(const float *Yp_dev, const int32_t *pos_dev, const float *topk_w_dev, const float *Ys_dev, bool shared,
            int T, int k, int d_h, int dtype, void *Y_dev, void *stream, const char *what) {
    if (T < 0 || k < 1 || d_h < 1) return MOE_EINVAL;
    if (dtype != MOE_DTYPE_BF16 && dtype != MOE_DTYPE_F32) return MOE_EINVAL;
    if (d_h % 4 != 0 || k > MOE_MAX_TOPK) return MOE_ESHAPE;
    if (T == 0) return MOE_OK;
    if (!Yp_dev || !pos_dev || !topk_w_dev || !Y_dev || (shared && !Ys_dev)) return MOE_EINVAL;
    if (!moe::aligned(Yp_dev, 16) || !moe::aligned(pos_dev, 4) || !moe::aligned(topk_w_dev, 4) ||
        !moe::aligned(Ys_dev, 16) || !moe::aligned(Y_dev, dtype == MOE_DTYPE_BF16 ? 8 : 16))
        return MOE_EINVAL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    // rows of d_h bf16 keep their 16-byte alignment when d_h is a multiple of 8
    const bool wide = dtype == MOE_DTYPE_BF16 && d_h % 8 == 0 && d_h >= kCombineWideMinCols && moe::aligned(Y_dev, 16) &&
                      static_cast<long long>(T) * d_h >= kCombineWide;
    const int cols = wide ? 2048 : 1024;
    const dim3 grid(T, (d_h + cols - 1) / cols);
    if (wide)
        hipLaunchKernelGGL((combine_kernel<true, 8>), grid, dim3(256), 0, st, Yp_dev, pos_dev, topk_w_dev, Ys_dev, k, d_h, Y_dev);
    else if (dtype == MOE_DTYPE_BF16)
        hipLaunchKernelGGL((combine_kernel<true, 4>), grid, dim3(256), 0, st, Yp_dev, pos_dev, topk_w_dev, Ys_dev, k, d_h, Y_dev);
    else
        hipLaunchKernelGGL((combine_kernel<false, 4>), grid, dim3(256), 0, st, Yp_dev, pos_dev, topk_w_dev, Ys_dev, k, d_h, Y_dev);
    return moe::check_launch(what);
}

}  // namespace

extern "C" int moe_combine(const float *Yp_dev, const int32_t *pos_dev, const float *topk_w_dev,
                           int T, int k, int d_h, int dtype, void *Y_dev, void *stream) {
    return combine(Yp_dev, pos_dev, topk_w_dev, nullptr, false, T, k, d_h, dtype, Y_dev, stream, "moe_combine");
}

extern "C" int moe_combine_shared(const float *Yp_dev, const int32_t *pos_dev, const float *topk_w_dev,
                                  const float *Ys_dev, int T, int k, int d_h, int dtype, void *Y_dev, void *stream) {
    return combine(Yp_dev, pos_dev, topk_w_dev, Ys_dev, true, T, k, d_h, dtype, Y_dev, stream, "moe_combine_shared");
}

extern "C" int moe_shared_dispatch(int T, int32_t *slot_off_dev, int32_t *perm_dev, int32_t *blocks_dev, void *stream) {
    if (T < 0 || !slot_off_dev || !blocks_dev || (T > 0 && !perm_dev)) return MOE_EINVAL;
    if (!moe::aligned(slot_off_dev, 4) || !moe::aligned(perm_dev, 4) || !moe::aligned(blocks_dev, 16)) return MOE_EINVAL;
    const int grid = T > 256 ? (T + 255) / 256 < 64 ? (T + 255) / 256 : 64 : 1;
    hipLaunchKernelGGL(shared_dispatch_kernel, dim3(grid), dim3(256), 0, static_cast<hipStream_t>(stream), T,
                       moe::ffn_block_rows(T), slot_off_dev, perm_dev, blocks_dev);
    return moe::check_launch("moe_shared_dispatch");
}
