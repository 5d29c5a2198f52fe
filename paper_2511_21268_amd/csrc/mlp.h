// Small MLP (8 -> 64 -> 64 -> 4, tanh hidden layers) that maps the features of
// one AMG level to the coefficients of its degree-4 polynomial smoother.
// Weights are held in BF16 on the device (used by forward and backward) with an
// FP32 master copy updated by Adam; all accumulation is FP32.  Every reduction
// over samples has a fixed order, so training is deterministic.
//
// Parameter vector (MLP_NPARAM entries):
//   W1[64][8] b1[64] W2[64][64] b2[64] W3[4][64] b3[4]
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.h"

namespace amgk {

constexpr int MLP_IN = 8, MLP_H = 64, MLP_OUT = 4;
constexpr int MLP_W1 = 0, MLP_B1 = MLP_W1 + MLP_H * MLP_IN, MLP_W2 = MLP_B1 + MLP_H,
              MLP_B2 = MLP_W2 + MLP_H * MLP_H, MLP_W3 = MLP_B2 + MLP_H, MLP_B3 = MLP_W3 + MLP_OUT * MLP_H,
              MLP_NPARAM = MLP_B3 + MLP_OUT;
constexpr int MLP_ACT = 2 * MLP_H;                    // stored activations per sample (h1, h2)
constexpr int MLP_DEL = MLP_OUT + 2 * MLP_H;          // workspace floats per sample

__device__ inline float bf16_to_f32(uint16_t b) { return __uint_as_float(((unsigned)b) << 16); }

// round to nearest even; NaN stays NaN
__device__ inline uint16_t f32_to_bf16(float f)
{
    unsigned u = __float_as_uint(f);
    if ((u & 0x7f800000u) == 0x7f800000u && (u & 0x007fffffu)) return (uint16_t)((u >> 16) | 0x40);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// A wave of the kernels below works on one hidden unit per lane (MLP_H = 64) and
// on four samples at a time: the lane's weights stay in registers, the samples'
// vectors are read from LDS by every lane at once, and four independent chains
// hide the latency of each.  Weights come as 16-byte loads with the alignment
// of a BF16 (the caller's array may start anywhere).
typedef unsigned vu4_bf16 __attribute__((ext_vector_type(4), aligned(2)));
constexpr int MLP_THREADS = 256, MLP_WAVES = MLP_THREADS / 64, MLP_TILE = 4;
constexpr int MLP_LD = MLP_H + 4;   // LDS row of one sample (16-byte aligned, rows on distinct banks)

// acc[k] += sum_j w[j] v[k][j] for the four samples' rows v[k] in LDS, j ascending
__device__ __forceinline__ void mlp_chain(float (&acc)[MLP_TILE], const float (&w)[MLP_H], const float *v)
{
#pragma unroll
    for (int j = 0; j < MLP_H; j += 4) {
        float4 t[MLP_TILE];
#pragma unroll
        for (int k = 0; k < MLP_TILE; k++) t[k] = *reinterpret_cast<const float4 *>(v + k * MLP_LD + j);
#pragma unroll
        for (int k = 0; k < MLP_TILE; k++) {
            acc[k] = fmaf(w[j], t[k].x, acc[k]);
            acc[k] = fmaf(w[j + 1], t[k].y, acc[k]);
            acc[k] = fmaf(w[j + 2], t[k].z, acc[k]);
            acc[k] = fmaf(w[j + 3], t[k].w, acc[k]);
        }
    }
}

// Y = W3 tanh(W2 tanh(W1 x + b1) + b2) + b3, every sum from its bias in
// ascending order.  Blocks of 16 samples.  Bound by latency (the weights from
// L2, two chains of 64 FMAs): 16,384 samples 76 -> 22 us, 58 samples
// 70 -> 6 us against one thread per sample, whose hidden vectors lived in
// scratch memory.
__global__ __launch_bounds__(MLP_THREADS) void k_mlp_fwd(const uint16_t *__restrict__ w, const float *__restrict__ X,
                                                         int B, float *__restrict__ Y, float *__restrict__ act)
{
    constexpr int S = MLP_WAVES * MLP_TILE;
    __shared__ float xs[S][MLP_IN], w3[MLP_OUT * MLP_H], w2s[MLP_H * (MLP_H + 1)];
    __shared__ __align__(16) float h1[S * MLP_LD], h2[S * MLP_LD];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6, r0 = wid * MLP_TILE;
    const int64_t s0 = (int64_t)blockIdx.x * S;
    if (tid < S * MLP_IN) {
        const int64_t s = s0 + tid / MLP_IN;
        xs[tid / MLP_IN][tid % MLP_IN] = s < B ? X[s * MLP_IN + tid % MLP_IN] : 0.0f;
    }
    w3[tid] = bf16_to_f32(w[MLP_W3 + tid]);
    static_assert(MLP_OUT * MLP_H == MLP_THREADS && S * MLP_IN <= MLP_THREADS, "one load per thread");
    float w1[MLP_IN], w2[MLP_H];
#pragma unroll
    for (int j = 0; j < MLP_IN; j++) w1[j] = bf16_to_f32(w[MLP_W1 + lane * MLP_IN + j]);
    // W2 in coalesced loads, its rows to the lanes through LDS
    for (int at = 8 * tid; at < MLP_H * MLP_H; at += 8 * MLP_THREADS) {
        const vu4_bf16 t = *reinterpret_cast<const vu4_bf16 *>(w + MLP_W2 + at);
#pragma unroll
        for (int h = 0; h < 4; h++) {
            float *to = w2s + (at / MLP_H) * (MLP_H + 1) + at % MLP_H + 2 * h;
            to[0] = __uint_as_float(t[h] << 16);
            to[1] = __uint_as_float(t[h] & 0xffff0000u);
        }
    }
    const float b1 = bf16_to_f32(w[MLP_B1 + lane]), b2 = bf16_to_f32(w[MLP_B2 + lane]);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < MLP_H; j++) w2[j] = w2s[lane * (MLP_H + 1) + j];
    float a[MLP_TILE];
#pragma unroll
    for (int k = 0; k < MLP_TILE; k++) {
        a[k] = b1;
#pragma unroll
        for (int j = 0; j < MLP_IN; j++) a[k] = fmaf(w1[j], xs[r0 + k][j], a[k]);
        a[k] = tanhf(a[k]);
        h1[(r0 + k) * MLP_LD + lane] = a[k];
        if (act && s0 + r0 + k < B) act[(s0 + r0 + k) * MLP_ACT + lane] = a[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < MLP_TILE; k++) a[k] = b2;
    mlp_chain(a, w2, h1 + r0 * MLP_LD);
#pragma unroll
    for (int k = 0; k < MLP_TILE; k++) {
        a[k] = tanhf(a[k]);
        h2[(r0 + k) * MLP_LD + lane] = a[k];
        if (act && s0 + r0 + k < B) act[(s0 + r0 + k) * MLP_ACT + MLP_H + lane] = a[k];
    }
    __syncthreads();
    // one output per thread of the first wave
    if (tid < S * MLP_OUT) {
        const int r = tid / MLP_OUT, o = tid % MLP_OUT;
        float y = bf16_to_f32(w[MLP_B3 + o]);
#pragma unroll 16
        for (int j = 0; j < MLP_H; j++) y = fmaf(w3[o * MLP_H + j], h2[r * MLP_LD + j], y);
        if (s0 + r < B) Y[s0 * MLP_OUT + tid] = y;
    }
}

// ---- gradient -----------------------------------------------------------------
//
// Loss L = mean over samples and outputs of (Y - T)^2; per sample
// dy = 2 (y - t) / (4 B), dh2 = W3^T dy * (1 - h2^2), dh1 = W2^T dh2 * (1 - h1^2).
// A block takes a chunk of the samples in tiles of 64: the deltas of a tile go
// to LDS, then every parameter's sum over the tile is added in registers -- W2's
// 64 x 64 sums dh2^T h1 on the matrix cores (v_mfma_f32_32x32x2_f32: FP32
// products and sums, one 32 x 32 quadrant per wave), the others one or two per
// lane.  The blocks' sums (MLP_PART floats each) are added in a fixed order by
// k_mlp_reduce; a single block writes gradient and loss itself.  Fixed orders throughout: training is deterministic.
// One thread per parameter walking all samples was bound by that serial chain:
// 16,384 samples 5,440 + 45 (deltas) -> 18 + 27 (k_mlp_reduce) us, 58 samples 18 + 39 -> 16
// us.
constexpr int MLP_ROWS = 64;              // samples per tile
constexpr int MLP_PART = MLP_NPARAM + 4;  // floats of one block's sums
constexpr int MLP_MAX_BLOCKS = 512;
constexpr int MLP_ONE_BLOCK = 2;          // most tiles of a batch that one block takes

// samples per block, and blocks: as many as the caller's workspace (MLP_DEL
// floats per sample) holds partial sums of, at most one per tile
struct MlpSplit {
    int chunk, blocks;
    explicit MlpSplit(int B)
    {
        const int64_t tiles = ((int64_t)B + MLP_ROWS - 1) / MLP_ROWS;
        int64_t n = (int64_t)B * MLP_DEL / MLP_PART;
        n = n < 1 ? 1 : n > MLP_MAX_BLOCKS ? MLP_MAX_BLOCKS : n;
        n = n > tiles ? tiles : n;
        const int64_t per = (tiles + n - 1) / n;   // tiles per block
        static_assert(MLP_ONE_BLOCK * MLP_ROWS * MLP_DEL >= 2 * MLP_PART, "two blocks past MLP_ONE_BLOCK tiles");
        chunk = (int)(per * MLP_ROWS);
        blocks = (int)((tiles + per - 1) / per);
    }
};

typedef float vf16 __attribute__((ext_vector_type(16)));

__global__ __launch_bounds__(MLP_THREADS) void k_mlp_back(const uint16_t *__restrict__ w, const float *__restrict__ X,
                                                          const float *__restrict__ act, const float *__restrict__ Y,
                                                          const float *__restrict__ T, int B, int chunk,
                                                          float *__restrict__ part, float *__restrict__ grad,
                                                          float *__restrict__ loss)
{
    __shared__ __align__(16) float h1s[MLP_ROWS * MLP_LD], h2s[MLP_ROWS * MLP_LD];
    __shared__ __align__(16) float d1s[MLP_ROWS * MLP_LD], d2s[MLP_ROWS * MLP_LD];
    __shared__ float xs[MLP_ROWS][MLP_IN], dys[MLP_ROWS][MLP_OUT], es[MLP_ONE_BLOCK * MLP_THREADS];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int64_t c0 = (int64_t)blockIdx.x * chunk, c1 = c0 + chunk < B ? c0 + chunk : B;
    const float scale = 2.0f / (float)((int64_t)MLP_OUT * B);
    // column `lane` of W2 and W3
    float w2[MLP_H], w3[MLP_OUT];
#pragma unroll
    for (int i = 0; i < MLP_H; i++) w2[i] = bf16_to_f32(w[MLP_W2 + i * MLP_H + lane]);
#pragma unroll
    for (int i = 0; i < MLP_OUT; i++) w3[i] = bf16_to_f32(w[MLP_W3 + i * MLP_H + lane]);
    // this lane's sums: W2 quadrant (wid / 2, wid % 2); W1[lane][2 wid], [2 wid
    // + 1]; W3[wid][lane]; one bias: b1 (wave 0), b2 (wave 1), b3 (wave 2)
    vf16 g2 = {};
    float g1a = 0.0f, g1b = 0.0f, g3 = 0.0f, gb = 0.0f;
    for (int64_t t0 = c0; t0 < c1; t0 += MLP_ROWS) {
        __syncthreads();   // the tile before is summed
        // the tile's inputs, zeros past the chunk: one dy per thread, x, and the
        // wave's samples' activations in registers
        constexpr int SW = MLP_ROWS / MLP_WAVES;   // samples per wave and tile
        static_assert(MLP_ROWS * MLP_OUT == MLP_THREADS, "one dy per thread");
        float h1[SW], h2[SW];
#pragma unroll
        for (int k = 0; k < SW; k++) {
            const int64_t s = t0 + wid * SW + k;
            h1[k] = s < c1 ? act[s * MLP_ACT + lane] : 0.0f;
            h2[k] = s < c1 ? act[s * MLP_ACT + MLP_H + lane] : 0.0f;
        }
        {
            const int64_t s = t0 + tid / MLP_OUT, at = t0 * MLP_OUT + tid;
            const float e = s < c1 ? Y[at] - T[at] : 0.0f;
            dys[tid / MLP_OUT][tid % MLP_OUT] = scale * e;
            if (gridDim.x == 1) es[at] = e;   // all of the batch, for the loss
        }
#pragma unroll
        for (int at = tid; at < MLP_ROWS * MLP_IN; at += MLP_THREADS)
            xs[at / MLP_IN][at % MLP_IN] = t0 + at / MLP_IN < c1 ? X[t0 * MLP_IN + at] : 0.0f;
        __syncthreads();
#pragma unroll
        for (int g = 0; g < SW; g += MLP_TILE) {
            const int r0 = wid * SW + g;
            float a[MLP_TILE];
#pragma unroll
            for (int k = 0; k < MLP_TILE; k++) {
                const int r = r0 + k;
                float d = 0.0f;
#pragma unroll
                for (int i = 0; i < MLP_OUT; i++) d = fmaf(w3[i], dys[r][i], d);
                // rows past the chunk add nothing, whatever the weights (inf * 0)
                d2s[r * MLP_LD + lane] = t0 + r < c1 ? d * (1.0f - h2[g + k] * h2[g + k]) : 0.0f;
                h1s[r * MLP_LD + lane] = h1[g + k];
                h2s[r * MLP_LD + lane] = h2[g + k];
                a[k] = 0.0f;
            }
            wave_lds_sync();   // these rows are this wave's own
            mlp_chain(a, w2, d2s + r0 * MLP_LD);
#pragma unroll
            for (int k = 0; k < MLP_TILE; k++)
                d1s[(r0 + k) * MLP_LD + lane] = t0 + r0 + k < c1 ? a[k] * (1.0f - h1[g + k] * h1[g + k]) : 0.0f;
        }
        __syncthreads();
        // W2: A = dh2^T (32 units x 2 samples), B = h1 (2 samples x 32 units)
        const float *pa = d2s + (lane >> 5) * MLP_LD + (wid >> 1) * 32 + (lane & 31);
        const float *pb = h1s + (lane >> 5) * MLP_LD + (wid & 1) * 32 + (lane & 31);
#pragma unroll 8
        for (int r = 0; r < MLP_ROWS; r += 2)
            g2 = __builtin_amdgcn_mfma_f32_32x32x2f32(pa[r * MLP_LD], pb[r * MLP_LD], g2, 0, 0, 0);
#pragma unroll 8
        for (int r = 0; r < MLP_ROWS; r++) {
            const float d1 = d1s[r * MLP_LD + lane];
            g1a = fmaf(d1, xs[r][2 * wid], g1a);
            g1b = fmaf(d1, xs[r][2 * wid + 1], g1b);
            g3 = fmaf(dys[r][wid], h2s[r * MLP_LD + lane], g3);
            gb += wid == 0 ? d1 : wid == 1 ? d2s[r * MLP_LD + lane] : dys[r][lane & (MLP_OUT - 1)];
        }
    }
    float *out = gridDim.x == 1 ? grad : part + (int64_t)blockIdx.x * MLP_PART;
    // accumulator register r of the 32 x 32 tile: row 8 (r / 4) + 4 (lane / 32) + r % 4, column lane % 32
#pragma unroll
    for (int r = 0; r < 16; r++) {
        const int i = (wid >> 1) * 32 + 8 * (r / 4) + 4 * (lane >> 5) + r % 4, j = (wid & 1) * 32 + (lane & 31);
        out[MLP_W2 + i * MLP_H + j] = g2[r];
    }
    out[MLP_W1 + lane * MLP_IN + 2 * wid] = g1a;
    out[MLP_W1 + lane * MLP_IN + 2 * wid + 1] = g1b;
    out[MLP_W3 + wid * MLP_H + lane] = g3;
    if (wid == 0) out[MLP_B1 + lane] = gb;
    else if (wid == 1) out[MLP_B2 + lane] = gb;
    else if (wid == 2 && lane < MLP_OUT) out[MLP_B3 + lane] = gb;
    if (tid == 0 && gridDim.x == 1 && loss) {
        float l = 0.0f;
#pragma unroll 8
        for (int v = 0; v < MLP_OUT * B; v++) l = fmaf(es[v], es[v], l);
        *loss = l / (float)(MLP_OUT * B);
    }
}

// The loss is the ascending FP32 chain l = fma(e, e, l) over all outputs, for
// every batch size (for a large batch that chain is some 1e-5 below the sum of
// its terms, the terms having shrunk to a few units of the sum's last place;
// callers compare losses of runs, so the value stays).  A single block walks it
// itself; here every thread runs 32 links of the chain,
// started from the FP64 sum of the terms before them, and the links' growth is
// added in FP64.  What a link rounds away depends on the running sum's binade,
// not on its low bits, so the segments together equal the chain to 1e-7.
constexpr int MLP_LOSS_THREADS = 1024, MLP_SEG = 32;
__device__ __forceinline__ void mlp_chain_loss(const float *__restrict__ Y, const float *__restrict__ T, int B,
                                               float *es /* threads * (MLP_SEG + 1) */, double *sums /* 32 */,
                                               float *__restrict__ loss)
{
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    constexpr int NW = MLP_LOSS_THREADS / 64;
    const int64_t n = (int64_t)B * MLP_OUT;
    double run = 0.0, grown = 0.0;
    for (int64_t t0 = 0; t0 < n; t0 += MLP_LOSS_THREADS * MLP_SEG) {
        __syncthreads();
#pragma unroll
        for (int k = 0; k < MLP_SEG; k++) {
            const int at = k * MLP_LOSS_THREADS + tid;   // one pad per segment: threads on distinct banks
            es[at + at / MLP_SEG] = t0 + at < n ? Y[t0 + at] - T[t0 + at] : 0.0f;
        }
        __syncthreads();
        const float *e = es + tid * (MLP_SEG + 1);
        double s = 0.0;
#pragma unroll
        for (int k = 0; k < MLP_SEG; k++) s = fma((double)e[k], (double)e[k], s);
        double upto = s;   // inclusive sum over the wave's lanes, then the waves before
        for (int o = 1; o < 64; o <<= 1) {
            const double t = __shfl_up(upto, o, 64);
            if (lane >= o) upto += t;
        }
        if (lane == 63) sums[wid] = upto;
        __syncthreads();
        double before = run;
        for (int v = 0; v < NW; v++) {
            if (v < wid) before += sums[v];
            run += sums[v];
        }
        const double below = __shfl_up(upto, 1, 64);
        const float l0 = (float)(lane ? before + below : before);
        float l = l0;
#pragma unroll
        for (int k = 0; k < MLP_SEG; k++) l = fmaf(e[k], e[k], l);
        // past an overflow the chain stays at infinity (or NaN)
        grown += isinf(l0) ? (double)l : (double)l - (double)l0;
    }
    grown = wave_sum(grown);
    __syncthreads();
    if (lane == 0) sums[wid] = grown;
    __syncthreads();
    if (tid != 0) return;
    double t = 0.0;
    for (int v = 0; v < NW; v++) t += sums[v];
    *loss = (float)t / (float)((int64_t)MLP_OUT * B);
}

// Sum of the blocks' partial sums: 64 parameters per block, 16 threads per
// parameter (each every 16th partial, ascending), then those in order; the
// last block forms the loss.
constexpr int MLP_RED = MLP_LOSS_THREADS / 64;
__global__ __launch_bounds__(MLP_LOSS_THREADS) void k_mlp_reduce(const float *__restrict__ part, int n,
                                                                 const float *__restrict__ Y,
                                                                 const float *__restrict__ T, int B,
                                                                 float *__restrict__ grad, float *__restrict__ loss)
{
    __shared__ float es[MLP_LOSS_THREADS * (MLP_SEG + 1)];
    __shared__ double sums[MLP_RED];
    if (blockIdx.x == gridDim.x - 1) {
        if (loss) mlp_chain_loss(Y, T, B, es, sums, loss);
        return;
    }
    const int lane = threadIdx.x & 63, seg = threadIdx.x >> 6, p = blockIdx.x * 64 + lane;
    float s = 0.0f;
    if (p < MLP_NPARAM) {
#pragma unroll 16
        for (int b = seg; b < n; b += MLP_RED) s += part[(int64_t)b * MLP_PART + p];
    }
    es[seg * 64 + lane] = s;
    __syncthreads();
    if (seg != 0 || p >= MLP_NPARAM) return;
    for (int v = 1; v < MLP_RED; v++) s += es[v * 64 + lane];
    grad[p] = s;
}

// gradient and loss of a batch; work: B * MLP_DEL floats
inline void mlp_gradient(const uint16_t *w, const float *X, const float *act, const float *Y, const float *T, int B,
                         float *work, float *grad, float *loss, hipStream_t st)
{
    const MlpSplit split(B);
    hipLaunchKernelGGL(k_mlp_back, dim3(split.blocks), dim3(MLP_THREADS), 0, st, w, X, act, Y, T, B, split.chunk, work,
                       grad, loss);
    if (split.blocks > 1)
        hipLaunchKernelGGL(k_mlp_reduce, dim3((MLP_NPARAM + 63) / 64 + 1), dim3(MLP_LOSS_THREADS), 0, st,
                           (const float *)work, split.blocks, Y, T, B, grad, loss);
}
inline void mlp_forward(const uint16_t *w, const float *X, int B, float *Y, float *act, hipStream_t st)
{
    // 16 threads a sample: a launch holds fewer than 2^28 samples
    constexpr int S = MLP_WAVES * MLP_TILE;
    constexpr int64_t MOST = int64_t(1) << 27;
    for (int64_t s0 = 0; s0 < B; s0 += MOST) {
        const int n = (int)(B - s0 < MOST ? B - s0 : MOST);
        hipLaunchKernelGGL(k_mlp_fwd, dim3((unsigned)((n + S - 1) / S)), dim3(MLP_THREADS), 0, st, w, X + s0 * MLP_IN, n,
                           Y + s0 * MLP_OUT, act ? act + s0 * MLP_ACT : nullptr);
    }
}

// Adam on the FP32 master weights, then the BF16 copy (round to nearest even).
__global__ void k_mlp_adam(float *__restrict__ master, uint16_t *__restrict__ w, const float *__restrict__ grad,
                           float *__restrict__ m, float *__restrict__ v, int step, float lr, float b1, float b2,
                           float eps)
{
    int p = blockIdx.x * 256 + threadIdx.x;
    if (p >= MLP_NPARAM) return;
    if (step > 0) {
        float g = grad[p];
        float mp = b1 * m[p] + (1.0f - b1) * g;
        float vp = b2 * v[p] + (1.0f - b2) * g * g;
        m[p] = mp;
        v[p] = vp;
        float mh = mp / (1.0f - powf(b1, (float)step));
        float vh = vp / (1.0f - powf(b2, (float)step));
        master[p] = master[p] - lr * mh / (sqrtf(vh) + eps);
    }
    w[p] = f32_to_bf16(master[p]);
}

}  // namespace amgk
