// a5: grouped expert FFN over the activated experts only (Janus Sec. 2.2: an expert is a
// fused gate/up GEMM and a down GEMM; at decode sizes the layer is bound by streaming the
// activated experts' weights from HBM, so latency follows the activated-expert count).
//
// This file: the weight packing, the workspace, the fp32 correctness path and the C entry
// point.  The bf16 kernels are in ffn_stream.hip.
//
// bf16 weights are consumed in a tile-packed layout: a 16-row x 32-column tile of a weight
// matrix is stored as the 1 KiB image of the MFMA A-operand of one wavefront (lane l holds row
// l%16, columns (l/16)*8 .. +7), and the two 16-row tiles a workgroup multiplies together (16
// gate + 16 up channels in stage 1, 32 output channels in stage 2) alternate per K-step, so a
// workgroup's share of a matrix is one contiguous run of 2 KiB steps read with fully coalesced
// 128-bit loads straight into MFMA registers.
//
// fp32 path (correctness configuration): tiles of 16 rows x 16 channels on the fp32 matrix cores, two launches.
#include <stdlib.h>

#include <mutex>

#include "dispatch_dev.h"

namespace {

// Workspace layout (bytes):
//   [0, kCtrlBytes)      control words, zeroed by moe_workspace_init and left zero by every call:
//                        int [1] = error word, then the per-block hand-off counters of the bf16
//                        kernels (see ffn_stream.hip)
//   [kCtrlBytes, ...)    act: SiLU(gate)*up of every local request row (fp32: [row][d_e];
//                        bf16: one region per entry of the work list, see ffn_stream.hip)
constexpr size_t kCtrlBytes = moe::kFfnCtrlBytes;

// ------------------------------------------------------------------ packing
// A matrix as pairs of 16-row tiles: dst [C][tiles][KS][2][64 lanes][8] from rows (slot, tile, half) of `cols` columns;
// row of a tile's half h: s*rows_per_slot + h*half_stride + tile*tile_stride.
//   W13 [C, 2*d_e, d_h] -> halves gate, up:   tile_stride 16, half_stride d_e
//   W2  [C, d_h, d_e]   -> rows 0-15, 16-31:  tile_stride 32, half_stride 16
// A copy: a wavefront moves STEPS K-steps of both halves of a tile pair (four: both 64-byte halves of each source line, 2 KiB
// of contiguous stores per K-step); the wavefronts of a slot are dealt over its K-steps and tiles alike, so that a matrix of
// few tiles or few K-steps still has its wavefronts everywhere.  At C = 17, d_h = 2048, d_e = 1408 (588 MB moved) 107 us for
// both matrices (5.5 TB/s with part of the source in the last-level cache from the call before; a plain device copy reaches
// 4.95) against 134 for a flat index of 16-byte pieces taken apart with 64-bit divisions; at C = 36, d_h = 7168, d_e = 2048
// 1136 against 1537 us.  The stores carry the streaming hint (132 us without); on the loads it costs the other half of each
// line (147 us).
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
constexpr int kPackWaves = 4;
template <int STEPS>
__global__ __launch_bounds__(kPackWaves * MOE_WAVE)
void pack_kernel(const u32x4 *__restrict__ src, u32x4 *__restrict__ dst, int tiles, int chunks, int cols, int rows_per_slot,
                 int tile_stride, int half_stride) {
    const int s = blockIdx.y;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / MOE_WAVE), lane = moe::lane_id();
    const int KS = cols / 32;
    const int unit = blockIdx.x * kPackWaves + wave;
    if (unit >= tiles * chunks) return;
    const int tile = unit / chunks, k0 = (unit - tile * chunks) * STEPS;
    const size_t row0 = static_cast<size_t>(s) * rows_per_slot + static_cast<size_t>(tile) * tile_stride + (lane & 15);
    u32x4 v[STEPS][2];
#pragma unroll
    for (int u = 0; u < STEPS; ++u) {
        const size_t kk = k0 + u < KS ? k0 + u : KS - 1;              // past the last K-step: that one again, not stored
#pragma unroll
        for (int h = 0; h < 2; ++h)
            v[u][h] = src[(row0 + static_cast<size_t>(h) * half_stride) * (cols / 8) + (lane >> 4) + kk * 4];
    }
    u32x4 *out = dst + ((static_cast<size_t>(s) * tiles + tile) * KS + k0) * 2 * MOE_WAVE + lane;
#pragma unroll
    for (int u = 0; u < STEPS; ++u)
        if (k0 + u < KS) {
#pragma unroll
            for (int h = 0; h < 2; ++h) __builtin_nontemporal_store(v[u][h], out + (u * 2 + h) * MOE_WAVE);
        }
}

// Four K-steps a wavefront when that gives every SIMD four of them, else one (C = 4, d_h = 64, d_e = 4096 and the other way round
// 5.4 us, 14 with a workgroup per tile pair; C = 1, d_h = 7168, d_e = 2048 29, 35).
constexpr long long kPackFour = 4096;
void launch_pack(const void *src, void *dst, int C, int tiles, int cols, int rows_per_slot, int tile_stride, int half_stride,
                 hipStream_t st) {
    const int KS = cols / 32, four = (KS + 3) / 4;
    const bool wide = KS >= 4 && static_cast<long long>(C) * tiles * four >= kPackFour;
    const int chunks = wide ? four : KS;
    const int gx = (tiles * chunks + kPackWaves - 1) / kPackWaves;
    const dim3 grid(gx, C), threads(kPackWaves * MOE_WAVE);
    const auto *in = static_cast<const u32x4 *>(src);
    auto *out = static_cast<u32x4 *>(dst);
    if (wide) hipLaunchKernelGGL(pack_kernel<4>, grid, threads, 0, st, in, out, tiles, chunks, cols, rows_per_slot, tile_stride, half_stride);
    else hipLaunchKernelGGL(pack_kernel<1>, grid, threads, 0, st, in, out, tiles, chunks, cols, rows_per_slot, tile_stride, half_stride);
}

__global__ void fill_zero_kernel(int *p, int n) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = 0;
}

// ------------------------------------------------------------------ fp32 path
// Tiles of 16 request rows of one slot x 16 channels (stage 1: the gate and the up rows of them) on the fp32 matrix cores:
// v_mfma_f32_16x16x4_f32, weights as the A operand (lane l: channel l%16), token rows as the B operand (lane l: row l%16), both
// read 16 bytes a lane, columns (l/16)*4 .. +3 of a K-step of 16; the four MFMAs of a K-step take one element of each.  The
// eight wavefronts of a workgroup split the K-steps round-robin and meet in LDS.  Few dependent loads bound these launches
// (slot offsets, request ids, operands), so a wavefront has two or four K-steps of all operands in flight.  With a wavefront per output
// and a workgroup per four outputs of a row, 16384 workgroups, half of which found no row, and every row read its expert again:
// T = 64, k = 2, d_h = 256, d_e = 512 11.2 + 5.2 us, 5.6 + 5.1 so; a layer step at T = 300, d_h = d_e = 640 127 us, 42 so.
// The matrix instruction is a chain of four fused multiply-adds, each rounded; the chains of a K-step, the K-steps and the groups
// are added pairwise and the wavefronts' sums in 64 bits, so that the error against 64 bits is a tenth smaller than with
// a chain per lane and a tree over the lanes (relative, of a layer: 1.37e-7 and 1.54e-7 there, 1.48e-7 and 1.63e-7 at 640 x 640).
typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int kF32Rows = 16, kF32Channels = 16, kF32Step = 16;
constexpr int kF32Waves = 8;

struct RowTile { int slot, row0, row_end; };
// Row tile b of the slots' row tiles in slot order; slot -1 past the last.  Uniform over the wavefront.
__device__ __forceinline__ RowTile find_row_tile(const int32_t *slot_off, int C, int b, int lane) {
    for (int s0 = 0; s0 < C; s0 += MOE_WAVE) {
        const int s = s0 + lane;
        const int lo = slot_off[s < C ? s : C], hi = slot_off[s < C ? s + 1 : C];
        const int n = (hi - lo + kF32Rows - 1) / kF32Rows;
        const int incl = moe::wave_incl_scan_i32(n);
        const int total = __builtin_amdgcn_readlane(incl, MOE_WAVE - 1);
        if (b < total) {
            const int src = __builtin_ctzll(__ballot(incl > b));
            const int row0 = __builtin_amdgcn_readlane(lo, src) + (b - __builtin_amdgcn_readlane(incl - n, src)) * kF32Rows;
            return {s0 + src, row0, __builtin_amdgcn_readlane(hi, src)};
        }
        b -= total;
    }
    return {-1, 0, 0};
}

// grid (channel tiles, bound of the row tiles).  GATED: A rows c and c + d_out of the slot, B rows through perm, out = SiLU(gate)*up;
// otherwise A rows c, B rows as they are.
template <bool GATED>
__global__ __launch_bounds__(kF32Waves * MOE_WAVE, 4)                 // two workgroups a CU
void ffn_f32_kernel(const float *__restrict__ B, const float *__restrict__ Wt, const int32_t *__restrict__ slot_off,
                    const int32_t *__restrict__ perm, float *__restrict__ out, int C, int k, int d_in, int d_out) {
    constexpr int F = GATED ? 2 : 1;
    constexpr int kAhead = GATED ? 2 : 4;                            // K-steps of all operands in flight
    __shared__ float part[F][kF32Waves][kF32Rows * kF32Channels];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / MOE_WAVE), lane = moe::lane_id();
    const RowTile rt = find_row_tile(slot_off, C, blockIdx.y, lane);
    if (rt.slot < 0) return;
    int row = rt.row0 + (lane & 15);
    row = row < rt.row_end ? row : rt.row_end - 1;                   // rows past the end repeat the last one, not stored
    const int c0 = blockIdx.x * kF32Channels;
    const int c = c0 + (lane & 15) < d_out ? c0 + (lane & 15) : d_out - 1;
    const int col = (lane >> 4) * 4;
    const float *wp = Wt + (static_cast<size_t>(rt.slot) * (F * d_out) + c) * d_in + col;
    const float *bp = B + static_cast<size_t>(GATED ? perm[row] / k : row) * d_in + col;
    const int steps = (d_in + kF32Step - 1) / kF32Step;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    f32x4 sum[F];
#pragma unroll
    for (int f = 0; f < F; ++f) sum[f] = zero;
    for (int s0 = wave; s0 < steps; s0 += kF32Waves * kAhead) {
        f32x4 a[kAhead][F], b[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int o = (s0 + u * kF32Waves) * kF32Step;
            const bool on = o + col < d_in;                          // d_in is a multiple of 4: whole pieces; past the end zeros
            const int at = on ? o : 0;
#pragma unroll
            for (int f = 0; f < F; ++f) {
                a[u][f] = *reinterpret_cast<const f32x4 *>(wp + static_cast<size_t>(f) * d_out * d_in + at - (on ? 0 : col));
                if (!on) a[u][f] = zero;
            }
            b[u] = *reinterpret_cast<const f32x4 *>(bp + at - (on ? 0 : col));
            if (!on) b[u] = zero;
        }
        f32x4 acc[F][kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
#pragma unroll
            for (int f = 0; f < F; ++f) acc[f][u] = zero;
            if (s0 + u * kF32Waves < steps) {                        // wave-uniform
#pragma unroll
                for (int f = 0; f < F; ++f) {
                    f32x4 m[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) m[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][f][i], b[u][i], zero, 0, 0, 0);
                    acc[f][u] = (m[0] + m[1]) + (m[2] + m[3]);
                }
            }
        }
#pragma unroll
        for (int f = 0; f < F; ++f) {
            if constexpr (kAhead == 4) sum[f] += (acc[f][0] + acc[f][1]) + (acc[f][2] + acc[f][3]);
            else sum[f] += acc[f][0] + acc[f][1];
        }
    }
    // lane l holds channels (l/16)*4 .. +3 of row l%16
#pragma unroll
    for (int f = 0; f < F; ++f) *reinterpret_cast<f32x4 *>(&part[f][wave][lane * 4]) = sum[f];
    __syncthreads();
    const int v = threadIdx.x;
    if (v >= kF32Rows * kF32Channels) return;
    float y[F];
#pragma unroll
    for (int f = 0; f < F; ++f) {
        double p = part[f][0][v];                                    // one rounding instead of seven
#pragma unroll
        for (int w = 1; w < kF32Waves; ++w) p += part[f][w][v];
        y[f] = static_cast<float>(p);
    }
    const int r = rt.row0 + ((v >> 2) & 15), ch = c0 + (v >> 6) * 4 + (v & 3);
    if (r < rt.row_end && ch < d_out)
        out[static_cast<size_t>(r) * d_out + ch] = GATED ? y[0] / (1.0f + expf(-y[0])) * y[F - 1] : y[0];
}

}  // namespace

namespace {
__global__ void set_word_kernel(int *p, int v) { *p = v; }
}  // namespace

extern "C" int moe_workspace_set_option(void *workspace_dev, size_t workspace_bytes, int option, int value, void *stream) {
    if (!workspace_dev || !moe::aligned(workspace_dev, 256)) return MOE_EINVAL;
    if (workspace_bytes < kCtrlBytes) return MOE_EWORKSPACE;
    if (value < 0) return MOE_EINVAL;
    int word;
    if (option == MOE_WS_OPT_SPIN_LIMIT) word = moe::kCtrlSpinLimit;
    else if (option == MOE_WS_OPT_WIDE_MIN_WORKGROUPS) word = moe::kCtrlWideMin;
    else return MOE_EINVAL;
    hipLaunchKernelGGL(set_word_kernel, dim3(1), dim3(1), 0, static_cast<hipStream_t>(stream),
                       static_cast<int *>(workspace_dev) + word, value);
    return moe::check_launch("moe_workspace_set_option");
}

// From this many tokens on the size counts a row of d_e bf16 per request more than the launches use: it is what callers have
// allocated by and what decides which shapes moe_grouped_ffn_static takes, so it stays as it is.
constexpr int kRowsTokens = 2048;

extern "C" size_t moe_workspace_bytes(int T, int k, int C, int d_h, int d_e, int dtype) {
    (void)d_h;
    if (T < 0 || k < 1 || C < 1 || d_e < 1) return 0;
    // fp32: one row per request; bf16: whole blocks of rows (at most C partly filled ones)
    const size_t bytes = dtype == MOE_DTYPE_F32
        ? static_cast<size_t>(T) * k * d_e * 4
        : moe::ffn_stream_act_bytes(T, k, C, d_e) + (T >= kRowsTokens ? static_cast<size_t>(T) * k * d_e * 2 : 0);
    return kCtrlBytes + (bytes + 255) / 256 * 256 + 256;
}

extern "C" int moe_workspace_init(void *workspace_dev, size_t workspace_bytes, void *stream) {
    if (!workspace_dev || !moe::aligned(workspace_dev, 256)) return MOE_EINVAL;
    if (workspace_bytes < kCtrlBytes) return MOE_EWORKSPACE;
    hipLaunchKernelGGL(fill_zero_kernel, dim3(64), dim3(256), 0, static_cast<hipStream_t>(stream),
                       static_cast<int *>(workspace_dev), static_cast<int>(kCtrlBytes / 4));
    return moe::check_launch("moe_workspace_init");
}

extern "C" int moe_workspace_status(const void *workspace_dev, int *status_host) {
    if (!workspace_dev || !status_host) return MOE_EINVAL;
    int hdr[2] = {0, 0};
    hipError_t e = hipMemcpy(hdr, workspace_dev, sizeof(hdr), hipMemcpyDeviceToHost);
    if (e != hipSuccess) { moe::set_hip_error(e, "moe_workspace_status"); return MOE_EHIP; }
    *status_host = hdr[moe::kCtrlStatus];
    return MOE_OK;
}

extern "C" int moe_pack_weights_bf16(const void *W13_dev, const void *W2_dev, int C, int d_h, int d_e,
                                     void *W13_packed_dev, void *W2_packed_dev, void *stream) {
    if (C < 1 || d_h < 1 || d_e < 1) return MOE_EINVAL;
    if (C > MOE_MAX_SLOTS || d_h % 32 != 0 || d_e % 32 != 0) return MOE_ESHAPE;
    if (!W13_dev || !W2_dev || !W13_packed_dev || !W2_packed_dev) return MOE_EINVAL;
    if (!moe::aligned(W13_dev, 16) || !moe::aligned(W2_dev, 16) || !moe::aligned(W13_packed_dev, 16) ||
        !moe::aligned(W2_packed_dev, 16))
        return MOE_EINVAL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    launch_pack(W13_dev, W13_packed_dev, C, d_e / 16, d_h, 2 * d_e, 16, d_e, st);
    launch_pack(W2_dev, W2_packed_dev, C, d_h / 32, d_e, d_h, 32, 16, st);
    return moe::check_launch("moe_pack_weights_bf16");
}

namespace {

// The checks of one set of experts; MOE_OK with T == 0 means that nothing is to be done.
int check_ffn(const void *X_dev, const void *W13_dev, const void *W2_dev, int T, int k, int C, int d_h, int d_e, int dtype,
              const int32_t *slot_off_dev, const int32_t *perm_dev, const int32_t *blocks_dev, const float *Yp_dev,
              const void *workspace_dev, size_t workspace_bytes) {
    if (T < 0 || k < 1 || C < 1 || d_h < 1 || d_e < 1) return MOE_EINVAL;
    if (dtype != MOE_DTYPE_BF16 && dtype != MOE_DTYPE_F32) return MOE_EINVAL;
    if (C > MOE_MAX_SLOTS || k > MOE_MAX_TOPK) return MOE_ESHAPE;
    if (static_cast<long long>(T) * k > 0x7fffffffLL) return MOE_ESHAPE;
    if (dtype == MOE_DTYPE_BF16 && (d_h % 32 != 0 || d_e % 32 != 0)) return MOE_ESHAPE;
    if (dtype == MOE_DTYPE_F32 && (d_h % 4 != 0 || d_e % 4 != 0)) return MOE_ESHAPE;
    if (T == 0) return MOE_OK;
    if (!X_dev || !W13_dev || !W2_dev || !slot_off_dev || !perm_dev || !Yp_dev || !workspace_dev) return MOE_EINVAL;
    if (!moe::aligned(X_dev, 16) || !moe::aligned(W13_dev, 16) || !moe::aligned(W2_dev, 16) ||
        !moe::aligned(Yp_dev, 16) || !moe::aligned(workspace_dev, 256) || !moe::aligned(slot_off_dev, 4) ||
        !moe::aligned(perm_dev, 4))
        return MOE_EINVAL;
    if (dtype == MOE_DTYPE_BF16 && (!blocks_dev || !moe::aligned(blocks_dev, 16))) return MOE_EINVAL;
    if (workspace_bytes < moe_workspace_bytes(T, k, C, d_h, d_e, dtype)) return MOE_EWORKSPACE;
    return MOE_OK;
}

moe::FfnCall ffn_call(const void *X_dev, const void *W13_dev, const void *W2_dev, int k, int C, int d_e, const int32_t *perm_dev,
                      const int32_t *blocks_dev, float *Yp_dev, void *workspace_dev) {
    char *ws = static_cast<char *>(workspace_dev);
    return {X_dev, W13_dev, W2_dev, k, C, d_e, blocks_dev, perm_dev, reinterpret_cast<int *>(ws),
            reinterpret_cast<uint16_t *>(ws + kCtrlBytes), Yp_dev};
}

int grouped_ffn(const void *X_dev, const void *W13_dev, const void *W2_dev,
                int T, int k, int C, int d_h, int d_e, int dtype,
                const int32_t *slot_off_dev, const int32_t *perm_dev, const int32_t *blocks_dev,
                float *Yp_dev, void *workspace_dev, size_t workspace_bytes, void *stream) {
    const int bad = check_ffn(X_dev, W13_dev, W2_dev, T, k, C, d_h, d_e, dtype, slot_off_dev, perm_dev, blocks_dev, Yp_dev,
                              workspace_dev, workspace_bytes);
    if (bad != MOE_OK || T == 0) return bad;
    hipStream_t st = static_cast<hipStream_t>(stream);
    char *ws = static_cast<char *>(workspace_dev);
    if (dtype == MOE_DTYPE_BF16) {
        // the kernels address token rows with 32-bit byte offsets
        if (static_cast<long long>(T) * d_h * 2 > 0xffffffffLL) return MOE_ESHAPE;
        const int rc = moe::launch_ffn_stream(
            ffn_call(X_dev, W13_dev, W2_dev, k, C, d_e, perm_dev, blocks_dev, Yp_dev, workspace_dev), T, d_h, st);
        if (rc != MOE_OK) return rc;
    } else {
        const long long rows = static_cast<long long>(T) * k;
        if (rows > 65535) return MOE_ESHAPE;
        float *act = reinterpret_cast<float *>(ws + kCtrlBytes);
        const unsigned tiles = static_cast<unsigned>(C + rows / kF32Rows);    // at most one partly filled tile a slot
        const auto channels = [](int n) { return static_cast<unsigned>((n + kF32Channels - 1) / kF32Channels); };
        hipLaunchKernelGGL(ffn_f32_kernel<true>, dim3(channels(d_e), tiles), dim3(kF32Waves * MOE_WAVE), 0, st,
                           static_cast<const float *>(X_dev), static_cast<const float *>(W13_dev), slot_off_dev, perm_dev, act,
                           C, k, d_h, d_e);
        hipLaunchKernelGGL(ffn_f32_kernel<false>, dim3(channels(d_h), tiles), dim3(kF32Waves * MOE_WAVE), 0, st,
                           act, static_cast<const float *>(W2_dev), slot_off_dev, perm_dev, Yp_dev, C, k, d_e, d_h);
    }
    return moe::check_launch("moe_grouped_ffn");
}

// Scratch of moe_grouped_ffn_static: one copy per GPU, held until the process ends.  In host code
// this name is only a handle for hipGetSymbolAddress; the kernels get the address it returns.
constexpr size_t kStaticScratchBytes = MOE_FFN_STATIC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void *g_scratch_ptr[kMaxDevices];        // device address of `scratch` on each GPU, looked up once per GPU

// Address of this GPU's copy of the scratch array (the current device's), or null with the HIP error recorded.
void *static_scratch() {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess || dev < 0 || dev >= kMaxDevices) {
        moe::set_hip_error(e != hipSuccess ? e : hipErrorInvalidDevice, "moe_grouped_ffn_static: hipGetDevice");
        return nullptr;
    }
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            moe::set_hip_error(e != hipSuccess ? e : hipErrorInvalidSymbol, "moe_grouped_ffn_static: hipGetSymbolAddress");
            return nullptr;
        }
        g_scratch_ptr[dev] = p;
    }
    return g_scratch_ptr[dev];
}

}  // namespace

extern "C" int moe_grouped_ffn(const void *X_dev, const void *W13_dev, const void *W2_dev,
                               int T, int k, int C, int d_h, int d_e, int dtype,
                               const int32_t *slot_off_dev, const int32_t *perm_dev, const int32_t *blocks_dev,
                               float *Yp_dev, void *workspace_dev, size_t workspace_bytes, void *stream) {
    return grouped_ffn(X_dev, W13_dev, W2_dev, T, k, C, d_h, d_e, dtype, slot_off_dev, perm_dev, blocks_dev, Yp_dev,
                       workspace_dev, workspace_bytes, stream);
}

extern "C" int moe_grouped_ffn_shared(const void *X_dev, const void *W13_dev, const void *W2_dev,
                                      int T, int k, int C, int d_h, int d_e, int dtype,
                                      const int32_t *slot_off_dev, const int32_t *perm_dev, const int32_t *blocks_dev,
                                      float *Yp_dev, void *workspace_dev, size_t workspace_bytes,
                                      const void *W13s_dev, const void *W2s_dev, int d_s,
                                      const int32_t *s_slot_off_dev, const int32_t *s_perm_dev, const int32_t *s_blocks_dev,
                                      float *Ys_dev, void *s_workspace_dev, size_t s_workspace_bytes, void *stream) {
    int rc = check_ffn(X_dev, W13_dev, W2_dev, T, k, C, d_h, d_e, dtype, slot_off_dev, perm_dev, blocks_dev, Yp_dev,
                       workspace_dev, workspace_bytes);
    if (rc == MOE_OK)
        rc = check_ffn(X_dev, W13s_dev, W2s_dev, T, 1, 1, d_h, d_s, dtype, s_slot_off_dev, s_perm_dev, s_blocks_dev, Ys_dev,
                       s_workspace_dev, s_workspace_bytes);
    if (rc != MOE_OK || T == 0) return rc;
    if (workspace_dev == s_workspace_dev) return MOE_EINVAL;         // the two sets hand over through control lines of their own
    if (dtype == MOE_DTYPE_BF16 && static_cast<long long>(T) * d_h * 2 <= 0xffffffffLL) {
        const moe::FfnCall routed = ffn_call(X_dev, W13_dev, W2_dev, k, C, d_e, perm_dev, blocks_dev, Yp_dev, workspace_dev);
        const moe::FfnCall shared = ffn_call(X_dev, W13s_dev, W2s_dev, 1, 1, d_s, s_perm_dev, s_blocks_dev, Ys_dev, s_workspace_dev);
        if (moe::ffn_stream_takes_shared(routed, shared, T, d_h)) {
            moe::launch_ffn_stream_shared(routed, shared, T, d_h, static_cast<hipStream_t>(stream));
            return moe::check_launch("moe_grouped_ffn_shared");
        }
    }
    rc = grouped_ffn(X_dev, W13_dev, W2_dev, T, k, C, d_h, d_e, dtype, slot_off_dev, perm_dev, blocks_dev, Yp_dev,
                     workspace_dev, workspace_bytes, stream);
    if (rc != MOE_OK) return rc;
    return grouped_ffn(X_dev, W13s_dev, W2s_dev, T, 1, 1, d_h, d_s, dtype, s_slot_off_dev, s_perm_dev, s_blocks_dev, Ys_dev,
                       s_workspace_dev, s_workspace_bytes, stream);
}

extern "C" int moe_grouped_ffn_static(const void *X_dev, const void *W13_dev, const void *W2_dev,
                                      int T, int k, int C, int d_h, int d_e, int dtype,
                                      const int32_t *slot_off_dev, const int32_t *perm_dev, const int32_t *blocks_dev,
                                      float *Yp_dev, void *stream) {
    if (T < 0 || k < 1 || C < 1 || d_h < 1 || d_e < 1) return MOE_EINVAL;
    if (dtype != MOE_DTYPE_BF16 && dtype != MOE_DTYPE_F32) return MOE_EINVAL;
    if (static_cast<long long>(T) * k > 0x7fffffffLL) return MOE_ESHAPE;
    // the size the allocating entry point would ask its caller for must fit the fixed array
    const size_t need = moe_workspace_bytes(T, k, C, d_h, d_e, dtype);
    if (need == 0 || need > kStaticScratchBytes) return MOE_EWORKSPACE;
    if (T == 0) return MOE_OK;
    void *ws = static_scratch();
    if (!ws) return MOE_EHIP;
    // The array keeps what the last call on this GPU left: the header (status word, options) and the
    // hand-off lines of every block this call can have must start at zero.  A fill kernel, not a
    // memset node, so that the call can be captured into a graph.
    if (dtype == MOE_DTYPE_BF16) {
        const long long lines = 1 + moe::ffn_max_blocks(T, k, C);
        if (lines * 1024 > static_cast<long long>(kCtrlBytes)) return MOE_ESHAPE;
        hipLaunchKernelGGL(fill_zero_kernel, dim3(static_cast<unsigned>((lines + 3) / 4)), dim3(256), 0,
                           static_cast<hipStream_t>(stream), static_cast<int *>(ws), static_cast<int>(lines * 256));
    }
    return grouped_ffn(X_dev, W13_dev, W2_dev, T, k, C, d_h, d_e, dtype, slot_off_dev, perm_dev, blocks_dev, Yp_dev,
                       ws, kStaticScratchBytes, stream);
}
