// sne_eval.hip - accuracy of estimated normals against ground truth on the
// device: the metrics e_A and e_P(phi) of eq. ea_ep (Sec. IV-A).
//
// psi_k is the angle between the estimate and the ground truth at pixel k.
// The paper writes it as an arccos of the normalised dot product; here it is
// atan2(|n x g|, n . g), the same angle without the arccos's loss of
// precision near 0 and 180 degrees.  Two passes: a grid-stride kernel
// reduces each block's pixels to (sum of psi, count, count of psi <= phi_j)
// in a scratch table, one block then reduces the table and writes
// e_A = mean psi, m and e_P(phi_j) = share of psi <= phi_j.
// The pass is bound by HBM reads: 12 B (FP32) or 6 B (FP16) of estimate,
// 12 B of ground truth and 1 B of mask per pixel.  64 x 480x640: FP32 79 us
// (6.2 TB/s), FP16 64 us (5.8 TB/s, the angles are 42 us of issue).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "sne_host.h"

namespace sne {
namespace {

constexpr int kEvalBlock = 256;
constexpr int kEvalWaves = kEvalBlock / kWave;

struct EvalArgs {
    const void *est;       // [B][3][hw] FP32 or FP16
    const float *gt;       // [B][3][hw] FP32
    const uint8_t *mask;   // [B][hw], or null: every pixel
    int64_t hw, nframes;   // pixels per frame, frames
    float phis[kEvalMaxPhis];
    int32_t nphi;
    double *partial;       // [gridDim.x][kEvalRow]
};

__device__ __forceinline__ float angle_deg(float ax, float ay, float az, float bx, float by,
                                           float bz) {
    const float cx = ay * bz - az * by;
    const float cy = az * bx - ax * bz;
    const float cz = ax * by - ay * bx;
    const float s = sqrtf(cx * cx + cy * cy + cz * cz);
    const float c = ax * bx + ay * by + az * bz;
    return atan2f(s, c) * 57.29577951308232f;
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
    return v;
}

// Plane groups, readable at any alignment: frames of a batch start wherever
// the frame before them ends, and the GPU's memory instructions take any
// address.
#define SNE_GLOBAL __attribute__((address_space(1)))
template <int OUT, int V> struct EstVec;
template <> struct EstVec<OUT_F32, 1> { typedef float T; };
template <> struct EstVec<OUT_F32, 4> {
    typedef float T __attribute__((ext_vector_type(4), aligned(4)));
};
template <> struct EstVec<OUT_F16, 1> { typedef _Float16 T; };
template <> struct EstVec<OUT_F16, 4> {
    typedef _Float16 T __attribute__((ext_vector_type(4), aligned(2)));
};
template <int V> struct MaskVec { typedef uint8_t T; };
template <> struct MaskVec<4> { typedef uint32_t T __attribute__((aligned(1))); };

template <typename T> __device__ __forceinline__ T load(const SNE_GLOBAL T *p) {
    return __builtin_nontemporal_load(p);  // read once
}
template <typename T> __device__ __forceinline__ float lane_of(const T &v, int k) {
    if constexpr (sizeof(T) >= 8) return (float)v[k];  // 4 x FP32 or 4 x FP16
    else return (float)v;
}

// What a missing mask reads as: every pixel of the group evaluated.
__device__ const uint8_t kAllValid[4] = {1, 1, 1, 1};

// Each thread takes V consecutive pixels of one frame at a time (V = 4: one
// 16-byte load per plane of FP32 data, 8 bytes of FP16, 4 bytes of mask),
// grid-stride over the frames' ceil(hw / V) groups; the last group of a frame
// ends at its last pixel and counts only what the group before left.  V = 4
// needs hw >= 4.
//
// The loop is uniform over a wave and the counts are kept once per wave, in
// scalar registers: a comparison and a scalar population count per pixel and
// threshold, where counts per lane took three vector instructions for each of
// kEvalMaxPhis.  NP is the number of thresholds counted, 4 or kEvalMaxPhis.
template <int OUT, int V, int NP>
__global__ __launch_bounds__(kEvalBlock) void eval_partial(EvalArgs a) {
    using ET = typename EstVec<OUT, V>::T;
    using GT = typename EstVec<OUT_F32, V>::T;
    using MT = typename MaskVec<V>::T;
    using EE = typename EstVec<OUT, 1>::T;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    double sum = 0.0;
    uint32_t cnt = 0, hit[kEvalMaxPhis] = {};  // per wave: far below 2^32
    const int64_t hwv = (a.hw + V - 1) / V;    // groups per frame
    const int64_t nv = a.nframes * hwv;
    const int64_t stride = (int64_t)gridDim.x * kEvalBlock;
    int64_t first = (int64_t)blockIdx.x * kEvalBlock + wave * kWave;  // of the wave
    // frame b and group q of the lane, advanced incrementally: the stride is
    // sb whole frames plus sq groups (no division per group, and one carry at
    // most however small the frames are)
    int64_t b = (first + lane) / hwv;
    int64_t q = first + lane - b * hwv;
    const int64_t sb = stride / hwv;
    const int64_t sq = stride - sb * hwv;
    const SNE_GLOBAL EE *est = (const SNE_GLOBAL EE *)a.est;
    const SNE_GLOBAL float *gt = (const SNE_GLOBAL float *)a.gt;
    const SNE_GLOBAL uint8_t *mask = (const SNE_GLOBAL uint8_t *)(a.mask ? a.mask : kAllValid);
    for (; first < nv; first += stride) {
        const bool in = first + lane < nv;
        // every load of the group at once (the planes are read whatever the
        // mask says); a lane past the end rereads the first group
        int64_t px = in ? q * V : 0;
        int skip = 0;  // of the group's V pixels, already counted
        if (V > 1 && px + V > a.hw) {
            skip = (int)(px + V - a.hw);
            px = a.hw - V;
        }
        const int64_t bb = in ? b : 0;
        const int64_t base = bb * 3 * a.hw + px;
        const MT mw = load((const SNE_GLOBAL MT *)(mask + (a.mask ? bb * a.hw + px : 0)));
        const ET ex = load((const SNE_GLOBAL ET *)(est + base));
        const ET ey = load((const SNE_GLOBAL ET *)(est + base + a.hw));
        const ET ez = load((const SNE_GLOBAL ET *)(est + base + 2 * a.hw));
        const GT gx = load((const SNE_GLOBAL GT *)(gt + base));
        const GT gy = load((const SNE_GLOBAL GT *)(gt + base + a.hw));
        const GT gz = load((const SNE_GLOBAL GT *)(gt + base + 2 * a.hw));
        b += sb;
        q += sq;
        if (q >= hwv) {
            q -= hwv;
            ++b;
        }
        // no branch on the mask: every pixel's angle is formed and the mask
        // selects what is counted (a branch would let the compiler sink the
        // plane loads behind the mask's round trip)
        const int from = in ? skip : V;
#pragma unroll
        for (int k = 0; k < V; ++k) {
            const bool ok = k >= from && ((mw >> (8 * k)) & 0xff) != 0;
            const float psi = angle_deg(lane_of(ex, k), lane_of(ey, k), lane_of(ez, k),
                                        lane_of(gx, k), lane_of(gy, k), lane_of(gz, k));
            sum += (double)(ok ? psi : 0.0f);
            const uint64_t okm = __ballot(ok);
            cnt += __builtin_popcountll(okm);
#pragma unroll
            for (int j = 0; j < NP; ++j)
                hit[j] += __builtin_popcountll(okm & __ballot(psi <= a.phis[j]));
        }
    }
    __shared__ double red[kEvalWaves][kEvalRow];
    sum = wave_sum(sum);
    if (lane == 0) {
        red[wave][0] = sum;
        red[wave][1] = cnt;
#pragma unroll
        for (int j = 0; j < kEvalMaxPhis; ++j) red[wave][2 + j] = hit[j];
    }
    __syncthreads();
    if (threadIdx.x < kEvalRow) {
        double v = 0.0;
#pragma unroll
        for (int w = 0; w < kEvalWaves; ++w) v += red[w][threadIdx.x];
        a.partial[(int64_t)blockIdx.x * kEvalRow + threadIdx.x] = v;
    }
}

// One block: sums the partial rows and writes {e_A, m, e_P(phi_0..)}.  It is
// latency, not work: the rows are read as pairs of columns, a whole number of
// rows per pass, so that a thread always meets the same pair (two sums
// instead of kEvalRow) and a pass of the block is one contiguous read; the
// columns then go to one wave per pair.  4.0 us for 2048 rows (6.0 with four
// waves that read a row per thread and reduced every column in each wave).
typedef double double2_t __attribute__((ext_vector_type(2)));
constexpr int kPairs = kEvalRow / 2;
constexpr int kFinalRows = 192;  // per pass
static_assert(kEvalRow % 2 == 0 && kFinalRows % kWave == 0, "rows are read in pairs of columns");
__global__ __launch_bounds__(kFinalRows * kPairs) void eval_final(const double *partial, int nrows,
                                                                   int nphi, double *result) {
    __shared__ double2_t red[kPairs][kFinalRows];
    __shared__ double tot[kEvalRow];
    const double2_t *src = reinterpret_cast<const double2_t *>(partial);
    const int col = threadIdx.x % kPairs, n = nrows * kPairs;
    double2_t acc = 0.0;
#pragma unroll 6
    for (int i = threadIdx.x; i < n; i += kFinalRows * kPairs) acc += src[i];
    red[col][threadIdx.x / kPairs] = acc;
    __syncthreads();
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    if (wave < kPairs) {
        double2_t t = red[wave][lane];
#pragma unroll
        for (int r = kWave; r < kFinalRows; r += kWave) t += red[wave][r + lane];
        const double x = wave_sum(t.x), y = wave_sum(t.y);
        if (lane == 0) {
            tot[2 * wave] = x;
            tot[2 * wave + 1] = y;
        }
    }
    __syncthreads();
    if (threadIdx.x < 2 + nphi) {
        const double m = tot[1];
        const double v = m > 0.0 ? tot[threadIdx.x] / m : 0.0;
        result[threadIdx.x] = threadIdx.x == 1 ? m : v;
    }
}

template <int OUT, int V> void launch_phis(const EvalArgs &a, int grid, hipStream_t s) {
    const dim3 g(grid), block(kEvalBlock);
    if (a.nphi <= 4) hipLaunchKernelGGL((eval_partial<OUT, V, 4>), g, block, 0, s, a);
    else hipLaunchKernelGGL((eval_partial<OUT, V, kEvalMaxPhis>), g, block, 0, s, a);
}
template <int OUT> void launch_partial(const EvalArgs &a, int grid, hipStream_t s) {
    if (a.hw >= 4) launch_phis<OUT, 4>(a, grid, s);
    else launch_phis<OUT, 1>(a, grid, s);
}

}  // namespace
}  // namespace sne

using namespace sne;

extern "C" {

int sne_accuracy(sne_ctx *ctx, const void *normals, int out_type, const float *gt,
                 const uint8_t *mask, int32_t B, int64_t frame_px, const float *phis_deg,
                 int32_t nphi, double *result, void *stream) {
    if (!ctx || B < 0 || frame_px < 0 || nphi < 0 || nphi > kEvalMaxPhis || !result ||
        (nphi > 0 && !phis_deg) || (out_type != SNE_OUT_F32 && out_type != SNE_OUT_F16))
        return SNE_ERR_ARG;
    const int64_t npx = (int64_t)B * frame_px;
    if (npx > 0 && (!normals || !gt)) return SNE_ERR_ARG;
    if (hipSetDevice(ctx->device) != hipSuccess) return SNE_ERR_HIP;
    hipStream_t st = (hipStream_t)stream;
    const int max_blocks = ctx->num_cu * 8;
    if (!ctx->d_eval) {
        if (hipMalloc(&ctx->d_eval, (size_t)max_blocks * kEvalRow * sizeof(double)) !=
                hipSuccess ||
            hipEventCreateWithFlags(&ctx->eval_done, hipEventDisableTiming) != hipSuccess)
            return SNE_ERR_HIP;
    } else if (hipStreamWaitEvent(st, ctx->eval_done, 0) != hipSuccess) {
        return SNE_ERR_HIP;  // the scratch table of an earlier call on another stream
    }
    int grid = 0;  // rows of partials written
    if (npx > 0) {
        EvalArgs a;
        a.est = normals;
        a.gt = gt;
        a.mask = mask;
        a.hw = frame_px;
        a.nframes = B;
        for (int j = 0; j < kEvalMaxPhis; ++j) a.phis[j] = j < nphi ? phis_deg[j] : -INFINITY;
        a.nphi = nphi;
        a.partial = ctx->d_eval;
        const int64_t units = frame_px >= 4 ? B * ((frame_px + 3) / 4) : npx;
        const int g = (int)std::max<int64_t>(
            1, std::min<int64_t>(max_blocks, (units + kEvalBlock - 1) / kEvalBlock));
        if (out_type == SNE_OUT_F16) launch_partial<OUT_F16>(a, g, st);
        else launch_partial<OUT_F32>(a, g, st);
        grid = g;
        if (hipGetLastError() != hipSuccess) return SNE_ERR_HIP;
    }
    hipLaunchKernelGGL(eval_final, dim3(1), dim3(kFinalRows * kPairs), 0, st,
                       ctx->d_eval, grid, nphi, result);
    if (hipGetLastError() != hipSuccess || hipEventRecord(ctx->eval_done, st) != hipSuccess)
        return SNE_ERR_HIP;
    return SNE_OK;
}

}  // extern "C"
