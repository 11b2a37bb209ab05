// mlp.hip -- the warm-start network of the learned IBM form: a
// 16 -> 64 -> 64 -> 3 multilayer perceptron with SiLU hidden activations,
// FP16 weights and FP32 accumulation; inference for every marker, and
// training (forward, backward and weight gradients in FP32 on the matrix cores,
// Adam) on samples the solver produced.
//
// Parameter layout (flat): W1[64][16] b1[64] W2[64][64] b2[64] W3[3][64] b3[3].
#include <hip/hip_runtime.h>

#include <algorithm>

#include "internal.hpp"
#include "mlp.hpp"

namespace turret {

// The logistic function with the hardware reciprocal (about 1 ulp), for
// FP16-operand inference, and with one Newton step more for training.
__device__ __forceinline__ float sigmoid_fast(float x) { return __builtin_amdgcn_rcpf(1.0f + __expf(-x)); }
__device__ __forceinline__ float sigmoidf(float x)
{
    const float v = 1.0f + __expf(-x), r = __builtin_amdgcn_rcpf(v);
    const float t = fmaf(fmaf(-v, r, 1.0f), r, r);
    return v > 3.0e38f ? 0.0f : t;   // (where exp overflows)
}

// ------------------------------------------------ inference on the matrix cores
// Inference runs on v_mfma_f32_16x16x16_f16: FP16 weights and activations,
// FP32 accumulation, SiLU in FP32.  A wavefront takes 16 samples at a time as
// the 16 columns of D = W X: for each layer the weights are the A operand
// (rows = output neurons, 16 per chunk) and the previous layer's activations
// the B operand (k = input neurons, 16 per step).  Lane l of the wave holds
// B[k][j] and D[i][j] for sample j = l % 16 and k, i = 4 (l / 16) + e
// (e = 0..3), so a layer's output chunk c is, as it stands in the registers,
// the next layer's operand for input step c.  The weights stay in registers
// while the wave strides over sample tiles.
typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
typedef float float4_t __attribute__((ext_vector_type(4)));

constexpr int kInSteps = (kMlpIn + 15) / 16;   // 16-wide input steps of layer 1 (zero padded)
constexpr int kHChunks = kMlpH / 16;
static_assert(kMlpH % 16 == 0 && kMlpOut <= 4, "layer sizes of the matrix-core inference");
static_assert(kMlpIn % 4 == 0 && kOffW2 % 4 == 0 && kOffB1 % 4 == 0 && kOffB2 % 4 == 0 && kOffW3 % 4 == 0,
              "8-byte aligned parameter blocks for the vector loads");

struct MlpRegs {
    half4_t w1[kHChunks][kInSteps], w2[kHChunks][kHChunks], w3[kHChunks];
    float b1[kHChunks][4], b2[kHChunks][4], b3[4];
};

// Four consecutive FP16 parameters starting at a multiple of 4 (one 8-byte load).
__device__ __forceinline__ half4_t load_half4(const _Float16 *th, int at)
{
    return *reinterpret_cast<const half4_t *>(th + at);
}

// The FP16 parameters, staged once per 256-thread workgroup in LDS with
// 16-byte copies (the parameter buffer extends to a 256-byte boundary, past
// the rounding up to 8 values).  Every load of a thread is issued before the
// first store, so the staging waits for one memory latency, not one per
// round of copies; the plain copy is padded to whole rounds (the padding
// holds repeats of the last vector) so that no store is conditional.
//
// W1 and W2 are also laid out in LDS as the register image of their A
// operands: slot (matrix, mc, kc) holds, for lanes l = 0..63 in a row, the 4
// values W[16 mc + l % 16][16 kc + 4 (l / 16) + 0..3], so that a wave takes
// each operand with one conflict-free 8-byte read per lane.  (Read straight
// from the row-major copy, the 16 rows of a W2 operand lie 128 bytes apart
// and fall into the same LDS banks.)  W3 and the biases are read from the
// plain copy, where lanes that share an address get it broadcast.
constexpr int kMlpParams8 = (kMlpParams + 7) / 8 * 8;
constexpr int kStageVecs = kMlpParams8 / 8;
constexpr int kStageRounds = (kStageVecs + 255) / 256;
constexpr int kStageHalves = kStageRounds * 256 * 8;
constexpr int kImgW1 = 0;                              // slot of (mc, kc): kImgW1 + mc kInSteps + kc
constexpr int kImgW2 = kHChunks * kInSteps;            // slot of (mc, kc): kImgW2 + mc kHChunks + kc
constexpr int kImgSlots = kImgW2 + kHChunks * kHChunks;
static_assert(kOffW2 % 8 == 0 && kOffB1 % 8 == 0 && kOffB2 % 8 == 0,
              "16-byte parameter vectors never straddle W1 / W2 and the next block");

struct MlpLds {
    _Float16 raw[kStageHalves];
    half4_t img[kImgSlots * 64];
};

// Places W[o][c..c+3] (c a multiple of 4) of a matrix with `steps` 16-wide
// column steps into its operand slot.
__device__ __forceinline__ void img_put(half4_t *img, int base, int steps, int o, int c, half4_t v)
{
    img[(base + (o >> 4) * steps + (c >> 4)) * 64 + (o & 15) + 16 * ((c & 15) >> 2)] = v;
}

__device__ inline void mlp_stage(const _Float16 *__restrict__ th, MlpLds &L)
{
    const uint4 *src = reinterpret_cast<const uint4 *>(th);
    uint4 *dst = reinterpret_cast<uint4 *>(L.raw);
    uint4 v[kStageRounds];
#pragma unroll
    for (int j = 0; j < kStageRounds; j++) v[j] = src[std::min((int)threadIdx.x + 256 * j, kStageVecs - 1)];
#pragma unroll
    for (int j = 0; j < kStageRounds; j++) {
        const int i = (int)threadIdx.x + 256 * j, h = 8 * i;
        dst[i] = v[j];
        const half4_t lo = __builtin_bit_cast(half4_t, make_uint2(v[j].x, v[j].y)),
                      hi = __builtin_bit_cast(half4_t, make_uint2(v[j].z, v[j].w));
        if (h < kOffB1) {
            const int o = (h - kOffW1) / kMlpIn, c = (h - kOffW1) % kMlpIn;
            img_put(L.img, kImgW1, kInSteps, o, c, lo);
            img_put(L.img, kImgW1, kInSteps, o, c + 4, hi);
        } else if (h >= kOffW2 && h < kOffB2) {
            const int o = (h - kOffW2) / kMlpH, c = (h - kOffW2) % kMlpH;
            img_put(L.img, kImgW2, kHChunks, o, c, lo);
            img_put(L.img, kImgW2, kHChunks, o, c + 4, hi);
        }
    }
    __syncthreads();
}

__device__ inline void mlp_load_regs(const MlpLds &L, MlpRegs &R)
{
    const _Float16 *th = L.raw;
    const int l = threadIdx.x & 63, r = l & 15, kq = (l >> 4) * 4;
    const _Float16 zero = (_Float16)0.0f;
#pragma unroll
    for (int mc = 0; mc < kHChunks; mc++) {
#pragma unroll
        for (int kc = 0; kc < kInSteps; kc++) R.w1[mc][kc] = L.img[(kImgW1 + mc * kInSteps + kc) * 64 + l];
#pragma unroll
        for (int kc = 0; kc < kHChunks; kc++) R.w2[mc][kc] = L.img[(kImgW2 + mc * kHChunks + kc) * 64 + l];
        // biases of the D rows this lane holds
        const half4_t b1 = load_half4(th, kOffB1 + 16 * mc + kq), b2 = load_half4(th, kOffB2 + 16 * mc + kq);
#pragma unroll
        for (int e = 0; e < 4; e++) {
            R.b1[mc][e] = (float)b1[e];
            R.b2[mc][e] = (float)b2[e];
        }
    }
#pragma unroll
    for (int kc = 0; kc < kHChunks; kc++) {
        const half4_t w = load_half4(th, kOffW3 + (r < kMlpOut ? r : 0) * kMlpH + 16 * kc + kq);
        const half4_t z = {zero, zero, zero, zero};
        R.w3[kc] = r < kMlpOut ? w : z;
    }
#pragma unroll
    for (int e = 0; e < 4; e++) R.b3[e] = kq + e < kMlpOut ? (float)th[kOffB3 + kq + e] : 0.0f;
}

__device__ __forceinline__ float4_t mfma16(half4_t a, half4_t b, float4_t c)
{
    return __builtin_amdgcn_mfma_f32_16x16x16f16(a, b, c, 0, 0, 0);
}

// One tile of 16 samples: x holds this lane's B operand of layer 1; the
// result holds, in lanes 0..15, outputs 0..kMlpOut-1 of sample l.  The bias
// is the accumulator's initial value, so the matrix cores add it.  SiLU is
// the tile's main cost: two quarter-rate transcendentals (exp, reciprocal)
// per hidden value.
__device__ inline float4_t mlp_tile(const MlpRegs &R, const half4_t x[kInSteps])
{
    half4_t a1[kHChunks], a2[kHChunks];
#pragma unroll
    for (int mc = 0; mc < kHChunks; mc++) {
        float4_t d = {R.b1[mc][0], R.b1[mc][1], R.b1[mc][2], R.b1[mc][3]};
#pragma unroll
        for (int kc = 0; kc < kInSteps; kc++) d = mfma16(R.w1[mc][kc], x[kc], d);
#pragma unroll
        for (int e = 0; e < 4; e++) a1[mc][e] = (_Float16)(d[e] * sigmoid_fast(d[e]));
    }
#pragma unroll
    for (int mc = 0; mc < kHChunks; mc++) {
        float4_t d = {R.b2[mc][0], R.b2[mc][1], R.b2[mc][2], R.b2[mc][3]};
#pragma unroll
        for (int kc = 0; kc < kHChunks; kc++) d = mfma16(R.w2[mc][kc], a1[kc], d);
#pragma unroll
        for (int e = 0; e < 4; e++) a2[mc][e] = (_Float16)(d[e] * sigmoid_fast(d[e]));
    }
    float4_t y = {R.b3[0], R.b3[1], R.b3[2], R.b3[3]};
#pragma unroll
    for (int kc = 0; kc < kHChunks; kc++) y = mfma16(R.w3[kc], a2[kc], y);
    return y;
}

// This lane's layer-1 operand for sample s of an n x kMlpIn FP32 array
// (zeros past n): four consecutive features per input step, one 16-byte
// load each.  The loads and the conversion to FP16 are split so that a
// wave can issue the next tile's loads before it works on the current tile.
static_assert(kMlpIn % 16 == 0, "one 16-byte feature load per lane and input step");
struct MlpRaw {
    float4 v[kInSteps];
};

__device__ inline MlpRaw mlp_load(const float *__restrict__ X, int s, int n)
{
    const int kq = ((threadIdx.x & 63) >> 4) * 4;
    MlpRaw r;
#pragma unroll
    for (int kc = 0; kc < kInSteps; kc++) {
        r.v[kc] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (s < n) r.v[kc] = *reinterpret_cast<const float4 *>(X + (long long)s * kMlpIn + 16 * kc + kq);
    }
    return r;
}

__device__ inline void mlp_convert(const MlpRaw &r, half4_t x[kInSteps])
{
#pragma unroll
    for (int kc = 0; kc < kInSteps; kc++) {
        x[kc][0] = (_Float16)r.v[kc].x;
        x[kc][1] = (_Float16)r.v[kc].y;
        x[kc][2] = (_Float16)r.v[kc].z;
        x[kc][3] = (_Float16)r.v[kc].w;
    }
}

// Tiles a wave takes per round.  Their features are loaded together, those
// of the first round before the weights are staged (both latencies overlap),
// those of the next round while the wave works on the current one.
constexpr int kMlpRound = 2;

// The inference loop shared by the two kernels: every wave strides over
// 16-sample tiles (the loop bounds are the same for the whole wave); epi(s,
// x, R) finishes sample s of this lane from its layer-1 operand x.
template <class Epi>
__device__ inline void mlp_stream(const _Float16 *__restrict__ th16, MlpLds &wsh, const float *__restrict__ X,
                                  int n, Epi &&epi)
{
    const int l = threadIdx.x & 63;
    const int wave = (int)(blockIdx.x * 4 + (threadIdx.x >> 6)), nwaves = (int)(gridDim.x * 4);   // 256 threads
    const int stride = 16 * nwaves;
    MlpRaw buf[kMlpRound];
#pragma unroll
    for (int j = 0; j < kMlpRound; j++) buf[j] = mlp_load(X, 16 * wave + j * stride + (l & 15), n);
    mlp_stage(th16, wsh);
    MlpRegs R;
    mlp_load_regs(wsh, R);
    for (int base = 16 * wave; base < n; base += kMlpRound * stride) {
#pragma unroll
        for (int j = 0; j < kMlpRound; j++) {
            const int s0 = base + j * stride;
            if (s0 >= n) break;
            half4_t x[kInSteps];
            mlp_convert(buf[j], x);
            buf[j] = mlp_load(X, s0 + kMlpRound * stride + (l & 15), n);   // the next round's tile j
            epi(s0 + (l & 15), x, R);
        }
    }
}

// Inference on caller arrays: X (n x kMlpIn) -> Y (n x 3).
__global__ void __launch_bounds__(256) k_mlp_forward(const _Float16 *__restrict__ th16, const float *__restrict__ X,
                                                     int n, float *__restrict__ Y)
{
    __shared__ __align__(16) MlpLds wsh;
    const int l = threadIdx.x & 63;
    mlp_stream(th16, wsh, X, n, [&](int s, const half4_t *x, const MlpRegs &R) {
        const float4_t y = mlp_tile(R, x);
        if (l < 16 && s < n)
#pragma unroll
            for (int j = 0; j < kMlpOut; j++) Y[(long long)s * kMlpOut + j] = y[j];
    });
}

// Warm start inside the IBM coupling: the network predicts, over the
// marker's feature scale s_k, the change of h from the previous step's final
// value: h = s_k (h(t-1) / s_k + MLP(features_k)), for every marker of an
// unmasked case; it becomes the first increment to spread.  A zero network
// starts from h(t-1), the control start.
__global__ void __launch_bounds__(256) k_mlp_warm_start(const _Float16 *__restrict__ th16, DevPtrs p, int Mtot)
{
    __shared__ __align__(16) MlpLds wsh;
    const int l = threadIdx.x & 63;
    mlp_stream(th16, wsh, p.feat, Mtot, [&](int k, const half4_t *x, const MlpRegs &R) {
        // the epilogue's operands, loaded before the matrix work
        bool live = false;
        float hp[3] = {0.0f, 0.0f, 0.0f};
        double hs = 0.0;
        if (l < 16 && k < Mtot) {
            live = p.body[p.mcase[k]].err == 0;
#pragma unroll
            for (int a = 0; a < 3; a++) hp[a] = p.feat[(long long)kMlpIn * k + kFeatHPrev + a];
            hs = p.hs[k];
        }
        const float4_t y = mlp_tile(R, x);
        if (live)
#pragma unroll
            for (int a = 0; a < 3; a++) {
                p.hk[3 * k + a] = 0.0;
                p.dh[3 * k + a] = ((double)hp[a] + (double)y[a]) * hs;
            }
    });
}

// ------------------------------------------------------------- training
// Forward, backward and the weight gradients in one pass, on
// v_mfma_f32_16x16x4_f32: FP32 operands (the FP16 weights widened) and FP32
// accumulation throughout.  A workgroup of 4 waves takes kTrainSamples samples at a time.
// Each wave runs 16 of them, the columns of every product, through the layers
// and back in registers: with step e of a 16-wide chunk taking input 4 g + e
// in lanes 16 g .. 16 g + 15, the rows a lane holds of one product are the
// operand it supplies to the next.  The weights are staged in LDS as operand
// images (one 16-byte read per lane and four steps, no bank conflicts).  The
// activations and errors then go to LDS, sample after sample in a row, and the
// weight gradients are products over the 64 samples: wave w forms rows 16 w ..
// 16 w + 15 of dW2 and dW1 and columns 16 w .. of dW3, kept in registers over
// all samples of the workgroup.  Sums run in a fixed order throughout, so the
// gradient is bitwise reproducible.
//
// Bound by latency (1.3 GFLOP at 8192 samples would take 10 us of the chip's
// FP32 rate over five gradients): one gradient took 214 us in four passes of
// one thread per sample or parameter through HBM scratch, and takes 17 us so
// (13 for this kernel).
typedef float row4_t __attribute__((ext_vector_type(4)));
// A caller's samples: rows at any float (the load is one instruction either way).
typedef float sample4_t __attribute__((ext_vector_type(4), aligned(4)));
constexpr int kTrainPitch = kTrainSamples + 4;   // floats per LDS row: 16-byte aligned, no bank conflicts

struct TrainLds {
    row4_t w1[kHChunks][64];                // [row tile][lane]: W1[16 t + i][4 g ..]
    row4_t w2[kHChunks][kHChunks][64];      // [row tile][chunk][lane]: W2[16 t + i][16 c + 4 g ..]
    row4_t w2t[kHChunks][kHChunks][64];     // the same of W2 transposed
    row4_t w3[kHChunks][64];                // [chunk][lane]: W3[i][16 c + 4 g ..], rows past the outputs 0
    float w3t[kMlpOut][kHChunks][64];       // [step][row tile][lane]: W3[e][16 t + i] for g = 0, else 0
    float b1[kMlpH], b2[kMlpH], b3[4];
    float x[kMlpIn][kTrainPitch], a1[kMlpH][kTrainPitch], a2[kMlpH][kTrainPitch];
    float z1[kMlpH][kTrainPitch], z2[kMlpH][kTrainPitch], dy[16][kTrainPitch];
    float loss[4];
};
static_assert(kMlpIn == 16 && kHChunks == 4, "one wave per 16 rows of the hidden layers, one chunk of inputs");

__device__ __forceinline__ float4_t mfma4(const row4_t &a, const row4_t &b, float4_t c)
{
#pragma unroll
    for (int e = 0; e < 4; e++) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[e], c, 0, 0, 0);
    return c;
}

__device__ inline void train_stage(const _Float16 *__restrict__ th, TrainLds &L)
{
    // four parameters per thread and round; all loads before the first store
    constexpr int kVecs = (kMlpParams + 3) / 4, kRounds = (kVecs + 255) / 256;
    half4_t v[kRounds];
#pragma unroll
    for (int j = 0; j < kRounds; j++) v[j] = load_half4(th, 4 * std::min((int)threadIdx.x + 256 * j, kVecs - 1));
    const row4_t zero = {0.0f, 0.0f, 0.0f, 0.0f};
    if (threadIdx.x < 64)
#pragma unroll
        for (int c = 0; c < kHChunks; c++) {
            if ((threadIdx.x & 15) >= kMlpOut) L.w3[c][threadIdx.x] = zero;
            if (threadIdx.x >= 16)
#pragma unroll
                for (int e = 0; e < kMlpOut; e++) L.w3t[e][c][threadIdx.x] = 0.0f;
        }
    if (threadIdx.x == 64) L.b3[3] = 0.0f;
    for (int k = threadIdx.x; k < (16 - kMlpOut) * kTrainPitch; k += 256) L.dy[kMlpOut + k / kTrainPitch][k % kTrainPitch] = 0.0f;
#pragma unroll
    for (int j = 0; j < kRounds; j++) {
        const int p = 4 * ((int)threadIdx.x + 256 * j);
        row4_t f;
#pragma unroll
        for (int e = 0; e < 4; e++) f[e] = (float)v[j][e];
        if (p < kOffB1) {
            const int o = p / kMlpIn, q = p % kMlpIn;
            L.w1[o >> 4][(o & 15) + 16 * (q >> 2)] = f;
        } else if (p < kOffW2) {
#pragma unroll
            for (int e = 0; e < 4; e++) L.b1[p - kOffB1 + e] = f[e];
        } else if (p < kOffB2) {
            const int o = (p - kOffW2) / kMlpH, q = (p - kOffW2) % kMlpH;
            L.w2[o >> 4][q >> 4][(o & 15) + 16 * ((q & 15) >> 2)] = f;
#pragma unroll
            for (int e = 0; e < 4; e++) L.w2t[q >> 4][o >> 4][((q & 15) + e) + 16 * ((o & 15) >> 2)][o & 3] = f[e];
        } else if (p < kOffW3) {
#pragma unroll
            for (int e = 0; e < 4; e++) L.b2[p - kOffB2 + e] = f[e];
        } else if (p < kOffB3) {
            const int o = (p - kOffW3) / kMlpH, q = (p - kOffW3) % kMlpH;
            L.w3[q >> 4][o + 16 * ((q & 15) >> 2)] = f;
#pragma unroll
            for (int e = 0; e < 4; e++) L.w3t[o][q >> 4][(q & 15) + e] = f[e];
        } else if (p < kMlpParams) {
#pragma unroll
            for (int e = 0; e < kMlpOut; e++) L.b3[e] = f[e];
        }
    }
    __syncthreads();
}

// SiLU of four pre-activations and its derivative.
__device__ __forceinline__ void silu4(const float4_t &z, row4_t &a, row4_t &d)
{
#pragma unroll
    for (int e = 0; e < 4; e++) {
        const float s = sigmoidf(z[e]);
        a[e] = z[e] * s;
        d[e] = s + a[e] * (1.0f - s);
    }
}

// Partial gradient and loss of the workgroup's samples into part[block] and
// loss_part[block].
__global__ void __launch_bounds__(256) k_mlp_train(const _Float16 *__restrict__ th16, const float *__restrict__ X,
                                                   const float *__restrict__ Tg, int n, MlpScratch sc)
{
    __shared__ __align__(16) TrainLds L;
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63, i = l & 15, g = l >> 4;
    const int col = 16 * w + i;   // this lane's sample of the round
    train_stage(th16, L);
    float4_t acc1 = {0.0f, 0.0f, 0.0f, 0.0f}, acc3 = acc1, acc2[kHChunks];
#pragma unroll
    for (int t = 0; t < kHChunks; t++) acc2[t] = acc1;
    float sb1 = 0.0f, sb2 = 0.0f, sb3 = 0.0f, loss = 0.0f;
    for (int base = kTrainSamples * blockIdx.x; base < n; base += kTrainSamples * gridDim.x) {
        const int s = base + col;
        const bool on = s < n;
        row4_t x = {0.0f, 0.0f, 0.0f, 0.0f}, dy = x;
        float tg[kMlpOut] = {};
        if (on) {
            x = *reinterpret_cast<const sample4_t *>(X + (long long)s * kMlpIn + 4 * g);
            if (g == 0)
#pragma unroll
                for (int e = 0; e < kMlpOut; e++) tg[e] = Tg[(long long)s * kMlpOut + e];
        }
        row4_t a1[kHChunks], d1[kHChunks], a2[kHChunks], d2[kHChunks];
#pragma unroll
        for (int t = 0; t < kHChunks; t++) {
            const float *b = L.b1 + 16 * t + 4 * g;
            const float4_t z = {b[0], b[1], b[2], b[3]};
            silu4(mfma4(L.w1[t][l], x, z), a1[t], d1[t]);
        }
#pragma unroll
        for (int t = 0; t < kHChunks; t++) {
            const float *b = L.b2 + 16 * t + 4 * g;
            float4_t z = {b[0], b[1], b[2], b[3]};
#pragma unroll
            for (int c = 0; c < kHChunks; c++) z = mfma4(L.w2[t][c][l], a1[c], z);
            silu4(z, a2[t], d2[t]);
        }
        float4_t y = {g == 0 ? L.b3[0] : 0.0f, g == 0 ? L.b3[1] : 0.0f, g == 0 ? L.b3[2] : 0.0f, 0.0f};
#pragma unroll
        for (int c = 0; c < kHChunks; c++) y = mfma4(L.w3[c][l], a2[c], y);
        if (on && g == 0)
#pragma unroll
            for (int e = 0; e < kMlpOut; e++) {
                const float r = y[e] - tg[e];
                dy[e] = r / (float)n;
                loss += r * r;
            }
        // back: dz2 = (W3^T dy) silu'(z2), dz1 = (W2^T dz2) silu'(z1)
#pragma unroll
        for (int t = 0; t < kHChunks; t++) {
            float4_t z = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int e = 0; e < kMlpOut; e++) z = __builtin_amdgcn_mfma_f32_16x16x4f32(L.w3t[e][t][l], dy[e], z, 0, 0, 0);
#pragma unroll
            for (int e = 0; e < 4; e++) {
                d2[t][e] *= z[e];
                L.z2[16 * t + 4 * g + e][col] = d2[t][e];
                L.a1[16 * t + 4 * g + e][col] = a1[t][e];
                L.a2[16 * t + 4 * g + e][col] = a2[t][e];
            }
        }
#pragma unroll
        for (int t = 0; t < kHChunks; t++) {
            float4_t z = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int c = 0; c < kHChunks; c++) z = mfma4(L.w2t[t][c][l], d2[c], z);
#pragma unroll
            for (int e = 0; e < 4; e++) L.z1[16 * t + 4 * g + e][col] = z[e] * d1[t][e];
        }
#pragma unroll
        for (int e = 0; e < 4; e++) L.x[4 * g + e][col] = x[e];
        if (g == 0)
#pragma unroll
            for (int e = 0; e < kMlpOut; e++) L.dy[e][col] = dy[e];
        __syncthreads();
        // the samples' part of the gradients
#pragma unroll
        for (int q = 0; q < kTrainSamples / 16; q++) {
            const int at = 16 * q + 4 * g;
            auto row = [&](const float (*m)[kTrainPitch], int r) { return *reinterpret_cast<const row4_t *>(&m[r][at]); };
            const row4_t z2 = row(L.z2, 16 * w + i), z1 = row(L.z1, 16 * w + i), d = row(L.dy, i);
#pragma unroll
            for (int t = 0; t < kHChunks; t++) acc2[t] = mfma4(z2, row(L.a1, 16 * t + i), acc2[t]);
            acc1 = mfma4(z1, row(L.x, i), acc1);
            acc3 = mfma4(d, row(L.a2, 16 * w + i), acc3);
            sb1 += (z1[0] + z1[1]) + (z1[2] + z1[3]);
            sb2 += (z2[0] + z2[1]) + (z2[2] + z2[3]);
            sb3 += (d[0] + d[1]) + (d[2] + d[3]);
        }
        __syncthreads();   // before the next round's stores
    }
    float *part = sc.part + (long long)blockIdx.x * kMlpParams;
#pragma unroll
    for (int e = 0; e < 4; e++) {
        const int o = 16 * w + 4 * g + e;
        part[kOffW1 + o * kMlpIn + i] = acc1[e];
#pragma unroll
        for (int t = 0; t < kHChunks; t++) part[kOffW2 + o * kMlpH + 16 * t + i] = acc2[t][e];
        if (g == 0 && e < kMlpOut) part[kOffW3 + e * kMlpH + 16 * w + i] = acc3[e];
    }
    // bias gradients: the four lanes of a row each hold a quarter of its samples
    auto quads = [&](float v) {
        v += __shfl_xor(v, 16);
        return v + __shfl_xor(v, 32);
    };
    sb1 = quads(sb1);
    sb2 = quads(sb2);
    sb3 = quads(sb3);
    if (g == 0) {
        part[kOffB1 + 16 * w + i] = sb1;
        part[kOffB2 + 16 * w + i] = sb2;
        if (w == 0 && i < kMlpOut) part[kOffB3 + i] = sb3;
    }
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) loss += __shfl_xor(loss, o);
    if (l == 0) L.loss[w] = loss;
    __syncthreads();
    if (threadIdx.x == 0) sc.loss_part[blockIdx.x] = ((L.loss[0] + L.loss[1]) + (L.loss[2] + L.loss[3])) * 0.5f / (float)n;
}

// Adam (Kingma & Ba): FP32 master weights and moments, and the FP16 copy used
// by the forward passes (round to nearest even).
struct AdamState {
    float *th32, *m, *v;
    _Float16 *th16;
    float lr, c1, c2;   // c = 1 - beta^step
};

__device__ inline void adam_update(const AdamState &A, int p, float g)
{
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    const float mm = b1 * A.m[p] + (1.0f - b1) * g;
    const float vv = b2 * A.v[p] + (1.0f - b2) * g * g;
    A.m[p] = mm;
    A.v[p] = vv;
    const float t = A.th32[p] - A.lr * (mm / A.c1) / (sqrtf(vv / A.c2) + eps);
    A.th32[p] = t;
    A.th16[p] = (_Float16)t;
}

// Gradient and loss from the workgroups' partial sums, and with ADAM the
// update instead of the gradient.  64 parameters per workgroup, 16 threads
// each: a serial sum over the partials was a chain of up to 256 loads.
template <bool ADAM>
__global__ void __launch_bounds__(1024) k_mlp_reduce(int nparts, MlpScratch sc, float *__restrict__ grad,
                                                     float *__restrict__ loss, AdamState A)
{
    __shared__ float sum[16][64];
    const int j = threadIdx.x & 63, k0 = threadIdx.x >> 6, p = blockIdx.x * 64 + j;
    float g = 0.0f;
    if (p < kMlpParams) {
#pragma unroll 4
        for (int k = k0; k < nparts; k += 16) g += sc.part[(long long)k * kMlpParams + p];
    }
    sum[k0][j] = g;
    __syncthreads();
    if (k0 == 0 && p < kMlpParams) {
#pragma unroll
        for (int k = 1; k < 16; k++) g += sum[k][j];
        if constexpr (ADAM) adam_update(A, p, g);
        else grad[p] = g;
    }
    if (blockIdx.x == 0 && k0 == 1 && loss) {
        float v = 0.0f;
        for (int k = j; k < nparts; k += 64) v += sc.loss_part[k];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
        if (j == 0) *loss = v;
    }
}

__global__ void k_mlp_round(const float *__restrict__ th32, _Float16 *__restrict__ th16)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p < kMlpParams) th16[p] = (_Float16)th32[p];
}

// ------------------------------------------------------------ launchers
// Workgroups of 4 waves for the matrix-core inference: one wave per 16-sample
// tile up to 2048 waves (2 per SIMD), which then stride.  Over the 161,818
// markers of the 64-case batch this takes 9.1 us; 1024 and 4096 waves were
// slower, and 8192 waves much slower (each workgroup stages the weights).
static dim3 infer_grid(int n)
{
    const int tiles = (n + 15) / 16;
    return dim3((unsigned)std::max(1, (std::min(tiles, 2048) + 3) / 4));
}

hipError_t launch_mlp_forward(const _Float16 *th16, const float *X, int n, float *Y, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_mlp_forward, infer_grid(n), dim3(256), 0, s, th16, X, n, Y);
    return hipGetLastError();
}

hipError_t launch_mlp_warm_start(const _Float16 *th16, const DevPtrs &p, int Mtot, hipStream_t s)
{
    if (Mtot <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_mlp_warm_start, infer_grid(Mtot), dim3(256), 0, s, th16, p, Mtot);
    return hipGetLastError();
}

hipError_t launch_mlp_grad(const _Float16 *th16, const float *X, const float *Tg, int n, const MlpScratch &sc,
                           float *grad, float *loss, hipStream_t s)
{
    const int nb = train_blocks(n);
    hipLaunchKernelGGL(k_mlp_train, dim3(nb), dim3(256), 0, s, th16, X, Tg, n, sc);
    hipLaunchKernelGGL(k_mlp_reduce<false>, dim3((kMlpParams + 63) / 64), dim3(1024), 0, s, nb, sc, grad, loss, AdamState{});
    return hipGetLastError();
}

hipError_t launch_mlp_train_step(float *th32, _Float16 *th16, float *m, float *v, const float *X, const float *Tg, int n,
                                 const MlpScratch &sc, float lr, int step, float *loss, hipStream_t s)
{
    const int nb = train_blocks(n);
    const AdamState A{th32, m, v, th16, lr, 1.0f - powf(0.9f, (float)step), 1.0f - powf(0.999f, (float)step)};
    hipLaunchKernelGGL(k_mlp_train, dim3(nb), dim3(256), 0, s, th16, X, Tg, n, sc);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;   // the parameters stay as they are
    hipLaunchKernelGGL(k_mlp_reduce<true>, dim3((kMlpParams + 63) / 64), dim3(1024), 0, s, nb, sc, nullptr, loss, A);
    return hipGetLastError();
}

hipError_t launch_mlp_round(const float *th32, _Float16 *th16, hipStream_t s)
{
    hipLaunchKernelGGL(k_mlp_round, dim3((kMlpParams + 255) / 256), dim3(256), 0, s, th32, th16);
    return hipGetLastError();
}

}  // namespace turret
