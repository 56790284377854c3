// Displacement CNN with FP8 e4m3 operands on the matrix cores, all four layers fused.
//
// The network and the pipeline are those of the BF16 pass (cnn_strips.h), with
// the operands of every layer in FP8 e4m3 (OCP format: 4 exponent bits, 3
// mantissa bits, largest finite value 448) and FP32 accumulation on
// v_mfma_f32_16x16x32_fp8_fp8, K = 32 per instruction as in the BF16 pass,
// half the bytes per operand.
//
// Scales, all powers of two so that applying them is exact:
//   * weights: one scale per output channel and layer, s_w = 2^ceil(log2(max|w| / 448));
//   * the velocity: s_v from max|u, v| over the grid (a reduction pass before the forward pass);
//   * the activations after layers 1-3: from a bound on their magnitude that follows from the
//     weights alone, |z_o| <= sum_{i,t} |w_oit| * A_in + |b_o| (with A_in the previous layer's
//     bound, and a margin of 1.25 for the rounding of the operands), so no value can overflow
//     the format whatever the input.
// A layer's accumulator starts at b_o / (s_w,o s_in) and is multiplied by s_w,o s_in / s_out
// before ReLU and rounding to e4m3 (round to nearest even) for the next layer; the last layer's
// nine tap products per output channel are summed in FP32 and multiplied by s_w,o s_in.
#include "cnn_strips.h"
#include "common.h"

namespace cnnsns {
namespace {

using namespace strips;

typedef long fp8x8;  // eight e4m3 values, the k = 8 (l/16) + j operand slots of lane l

// What the forward pass forms its scales from, written by k_fp8_scan
constexpr int kMaxBlocks = 160;  // what the workspace of 21.5 KiB has room for
struct Fp8Scales {
    float vmax[kMaxBlocks];   // max |u|, |v| over a block's share of the grid
    float s_w[4][C];          // weight scale per layer and output channel (layer 4: channels 0, 1)
    float rsum[3][C];         // sum of |w| over inputs and taps, layers 1..3
};
static_assert(sizeof(fp8x8) * PACKED + sizeof(Fp8Scales) <= 22016, "the workspace that the interface states");

__device__ __forceinline__ float pow2_at_least(float x)
{
    // the smallest power of two >= x (x > 0 and finite), else 1
    if (!(x > 0.f) || !(x < 3.0e38f)) return 1.f;
    int e;
    const float m = frexpf(x, &e);  // x = m 2^e, m in [0.5, 1)
    return ldexpf(1.f, m == 0.5f ? e - 1 : e);
}

__device__ __forceinline__ uint32_t to_e4m3_pair(float lo, float hi)
{
    return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(lo, hi, 0, false) & 0xffffu;
}

// One launch for what the pass needs of the weights and of the whole grid.  Blocks 0 .. 5: layer 1, the halves of 16
// output channels of layers 2 and 3, layer 4: each stages its FP32 weights in LDS, a wavefront reduces the max and the
// sum of |w| of an output channel, and all threads pack.  The others: max |u|, |v| of their share of the 2 G^2 velocity
// values.  The chain of activation bounds, which needs both, is a few instructions at the pass's start.  With a clear,
// one atomic maximum a block and a one-block kernel for weights and chain instead: 21 us at G = 64, 30 at 1531 and 61 at
// 4096; now 5, 5 and 20, and 2 us more in the pass.
constexpr int kScanThreads = 1024, kWeightBlocks = 6;
__global__ __launch_bounds__(kScanThreads) void k_fp8_scan(const float* __restrict__ w1, const float* __restrict__ w2,
                                                           const float* __restrict__ w3, const float* __restrict__ w4,
                                                           int64_t count, const float* __restrict__ vel,
                                                           Fp8Scales* __restrict__ s, fp8x8* __restrict__ packed)
{
    __shared__ float s_w[16 * C * 9];
    __shared__ float s_x[C];  // weight scale per output channel, or the wavefronts' maxima
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, b = blockIdx.x;
    if (b >= kWeightBlocks) {
        const int64_t step = (int64_t)(gridDim.x - kWeightBlocks) * kScanThreads;
        int64_t k = (int64_t)(b - kWeightBlocks) * kScanThreads + tid;
        // four at a time, from the first 16-byte boundary on; the values before it and past the last four one by one
        const int64_t head = std::min<int64_t>(count, (16 - ((uintptr_t)vel & 15)) % 16 / 4), quads = (count - head) / 4;
        const v4f* from = reinterpret_cast<const v4f*>(vel + head);
        float m = 0.f;
        if (k < head) m = fabsf(vel[k]);
        if (head + 4 * quads + k < count) m = fmaxf(m, fabsf(vel[head + 4 * quads + k]));
#pragma unroll 4
        for (; k < quads; k += step) {
            const v4f x = from[k];
            m = fmaxf(fmaxf(fmaxf(m, fabsf(x[0])), fmaxf(fabsf(x[1]), fabsf(x[2]))), fabsf(x[3]));
        }
        for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
        if (lane == 0) s_x[wave] = m;
        __syncthreads();
        if (tid == 0) {
            for (int w = 1; w < kScanThreads / 64; ++w) m = fmaxf(m, s_x[w]);
            s->vmax[b - kWeightBlocks] = m;
        }
        return;
    }
    const int layer = b == 0 ? 0 : b == 5 ? 3 : (b + 1) / 2, c0 = b == 2 || b == 4 ? 16 : 0;  // first channel
    const int channels = b == 0 ? C : b == 5 ? 2 : 16, per = (layer == 0 ? 2 : C) * 9;
    const float* w = (layer == 0 ? w1 : layer == 1 ? w2 : layer == 2 ? w3 : w4) + c0 * per;
    for (int k = tid; k < channels * per; k += kScanThreads) s_w[k] = w[k];
    __syncthreads();
    for (int o = wave; o < channels; o += kScanThreads / 64) {
        float mx = 0.f, sm = 0.f;
        for (int k = lane; k < per; k += 64) {
            const float a = fabsf(s_w[o * per + k]);
            mx = fmaxf(mx, a);
            sm += a;
        }
        for (int off = 32; off > 0; off >>= 1) {
            mx = fmaxf(mx, __shfl_xor(mx, off));
            sm += __shfl_xor(sm, off);
        }
        if (lane == 0) {
            s->s_w[layer][c0 + o] = s_x[o] = pow2_at_least(mx / 448.f);
            if (layer < 3) s->rsum[layer][c0 + o] = sm;
        }
    }
    __syncthreads();
    // layers 2 and 3: the half's fragments are every second one of the layer's
    fp8x8* to = packed + (layer == 0 ? 0 : layer == 3 ? P1 + 2 * P2 : P1 + (layer - 1) * P2);
    const int n = layer == 0 || layer == 3 ? 2 * 64 : 9 * 64;
    for (int e = tid; e < n; e += kScanThreads) {
        const int l = e & 63, i = l & 15, q = l >> 4;
        float v[8];
        if (layer == 0) {
            const int o = (e >> 6) * 16 + i;
            const float r = 1.f / s_x[o];
            for (int j = 0; j < 8; ++j) {
                const int k = 8 * q + j;
                v[j] = k < 18 ? s_w[(o * 2 + (k & 1)) * 9 + (k >> 1)] * r : 0.f;
            }
        } else if (layer < 3) {
            const float r = 1.f / s_x[i];
            for (int j = 0; j < 8; ++j) v[j] = s_w[(i * C + chan_at(8 * q + j)) * 9 + (e >> 6)] * r;
        } else {
            int o, tap;
            const bool used = conv4_row(16 * (e >> 6) + i, o, tap);
            const float r = 1.f / s_x[o];
            for (int j = 0; j < 8; ++j) v[j] = used ? s_w[(o * C + chan_at(8 * q + j)) * 9 + tap] * r : 0.f;
        }
        uint64_t word = 0;
        for (int j = 0; j < 8; j += 2) word |= (uint64_t)to_e4m3_pair(v[j], v[j + 1]) << (8 * j);
        to[layer == 0 || layer == 3 ? e : (2 * (e >> 6) + (c0 >> 4)) * 64 + l] = (fp8x8)word;
    }
}

struct Fp8 {
    using Op = fp8x8;
    static constexpr int BYTES = 32;
    struct Args {
        const Fp8Scales* sc;
        int maxima;  // of sc->vmax
        const float *b1, *b2, *b3, *b4;
    };
    v4f start[2][2], fac[2][2];
    float rv, out4, bo, sum0;

    // the layers' bounds and scales, lane % 32 = output channel, and of these the lane's constants
    __device__ __forceinline__ Fp8(const Args& a, bool first, int q, int oo) : bo(a.b4[oo]), sum0(0.f)
    {
        const float margin = 1.25f;  // covers the rounding of operands (at most 2^-4 each)
        const int lane = threadIdx.x & 63, o = lane & (C - 1);
        const float bl[3] = { a.b1[o], a.b2[o], a.b3[o] };
        float A = 0.f;
        for (int k = lane; k < a.maxima; k += 64) A = fmaxf(A, a.sc->vmax[k]);
        for (int off = 32; off > 0; off >>= 1) A = fmaxf(A, __shfl_xor(A, off));
        float s_in = pow2_at_least(A / 448.f), init[2], scale[2];
        rv = 1.f / s_in;
#pragma unroll
        for (int l = 0; l < 3; ++l) {
            float P = margin * a.sc->rsum[l][o] * A + fabsf(bl[l]);
            for (int off = 16; off > 0; off >>= 1) P = fmaxf(P, __shfl_xor(P, off));
            const float s_out = pow2_at_least(P / 448.f), sc = a.sc->s_w[l][o] * s_in;
            if (l == 0 || l == (first ? 1 : 2)) {
                init[l != 0] = bl[l] / sc;
                scale[l != 0] = sc / s_out;
            }
            A = P;
            s_in = s_out;
        }
        out4 = a.sc->s_w[3][oo] * s_in;
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int c = 16 * (k >> 2 & 1) + 4 * q + (k & 3);
            start[k >> 3][k >> 2 & 1][k & 3] = __shfl(init[k >> 3], c);
            fac[k >> 3][k >> 2 & 1][k & 3] = __shfl(scale[k >> 3], c);
        }
    }
    // A store of 16 consecutive pixels at one chunk, and a read of these at two, fall on distinct banks.
    static __device__ __forceinline__ int place(int p) { return (p >> 2) & 3; }
    static __device__ __forceinline__ v4f mfma(const Op& a, const Op& b, const v4f& c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(a, b, c, 0, 0, 0);
    }
    __device__ __forceinline__ uint32_t vel(float u, float v) const { return to_e4m3_pair(u * rv, v * rv); }
    static __device__ __forceinline__ Op gather(const uint32_t (&v)[4])
    {
        return (Op)((uint64_t)(v[0] | v[1] << 16) | (uint64_t)(v[2] | v[3] << 16) << 32);
    }
    // scaled to the next layer's operand scale, ReLU, rounded to e4m3
    template <int LAYER>
    __device__ __forceinline__ void act(const v4f& lo, const v4f& hi, uint32_t (&w)[2]) const
    {
        auto relu = [](float x) { return fmaxf(x, 0.f); };
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int r = 2 * k;
            w[k] = __builtin_amdgcn_cvt_pk_fp8_f32(relu(lo[r] * fac[LAYER][0][r]), relu(hi[r] * fac[LAYER][1][r]), 0, false);
            w[k] = __builtin_amdgcn_cvt_pk_fp8_f32(relu(lo[r + 1] * fac[LAYER][0][r + 1]),
                                                   relu(hi[r + 1] * fac[LAYER][1][r + 1]), w[k], true);
        }
    }
    __device__ __forceinline__ float sum(float s) const { return bo + out4 * s; }
};

__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_cnn_fp8(
    int32_t G, Plan plan, const float* __restrict__ vel, const fp8x8* __restrict__ packed, Fp8::Args a,
    float* __restrict__ disp)
{
    pass<Fp8>(G, plan, vel, packed, a, disp);
}

}  // namespace

size_t cnn_fp8_workspace_bytes()
{
    return sizeof(fp8x8) * (size_t)PACKED + ((sizeof(Fp8Scales) + 255) / 256) * 256;
}

void cnn_fp8_forward(int32_t G, const float* vel, const cnnsns_cnn& w, float* disp, void* ws, unsigned grid,
                     hipStream_t stream)
{
    fp8x8* packed = static_cast<fp8x8*>(ws);
    Fp8Scales* sc = reinterpret_cast<Fp8Scales*>(static_cast<char*>(ws) + sizeof(fp8x8) * (size_t)PACKED);
    const int64_t count = 2 * (int64_t)G * G;
    const int blocks = (int)std::min<int64_t>(kMaxBlocks, (count + 4 * kScanThreads - 1) / (4 * kScanThreads));
    k_fp8_scan<<<kWeightBlocks + blocks, kScanThreads, 0, stream>>>(w.w[0], w.w[1], w.w[2], w.w[3], count, vel, sc, packed);
    const Plan plan = strip_rows(G, (int)grid);
    k_cnn_fp8<<<(plan.blocks + 7) / 8 * 8, kThreads, 0, stream>>>(
        G, plan, vel, packed, Fp8::Args{ sc, blocks, w.b[0], w.b[1], w.b[2], w.b[3] }, disp);
    hip_check(hipGetLastError(), "fp8 cnn launch");
}

}  // namespace cnnsns
