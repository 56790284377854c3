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

// Scales and the per-channel epilogue factors, written by k_fp8_prep
struct Fp8Scales {
    unsigned vmax_bits;       // max |u|, |v| over the grid (bit pattern of a non-negative float)
    float s_v;                // velocity scale
    float s_a[3];             // activation scales after layers 1..3
    float s_w[4][C];          // weight scale per layer and output channel (layer 4: channels 0, 1)
    float init[3][C];         // accumulator start b_o / (s_w,o s_in) of layers 1..3
    float fac[3][C];          // s_w,o s_in / s_out of layers 1..3
    float out4[2];            // s_w4,o s_a3
};

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

__global__ void k_fp8_clear(Fp8Scales* s)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) s->vmax_bits = 0u;
}

// max |u|, |v| over the 2 G^2 velocity values: a block reduces its share through LDS and makes one
// atomic update (one per wavefront on a single word serialises thousands of updates)
constexpr int kMaxThreads = 512;
__global__ __launch_bounds__(kMaxThreads) void k_fp8_absmax(int64_t count, const float* __restrict__ vel, Fp8Scales* s)
{
    __shared__ float s_m[kMaxThreads / 64];
    float m = 0.f;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < count; k += (int64_t)gridDim.x * blockDim.x)
        m = fmaxf(m, fabsf(vel[k]));
    for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
    if ((threadIdx.x & 63) == 0) s_m[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kMaxThreads / 64; ++w) m = fmaxf(m, s_m[w]);
        atomicMax(&s->vmax_bits, __float_as_uint(m));
    }
}

// Weight scales, activation scales and the packed e4m3 weights; one block of 1024 threads.  The
// FP32 weights are staged in LDS (78 KiB), each wavefront reduces the max and the sum of |w| of
// its output channels, the first wavefront chains the layer bounds (one lane per channel), and
// all threads pack.
constexpr int NW1 = C * 2 * 9, NW23 = C * C * 9, NW4 = 2 * C * 9;
__global__ __launch_bounds__(1024) void k_fp8_prep(const float* __restrict__ w1, const float* __restrict__ w2,
                                                   const float* __restrict__ w3, const float* __restrict__ w4,
                                                   const float* __restrict__ b1, const float* __restrict__ b2,
                                                   const float* __restrict__ b3, Fp8Scales* s,
                                                   fp8x8* __restrict__ packed)
{
    __shared__ float s_w[NW1 + 2 * NW23 + NW4];
    __shared__ float s_rsum[3][C];   // sum of |w| over inputs and taps per output channel, layers 1..3
    __shared__ float s_scale[4][C];  // weight scale per layer and output channel
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    float* const sw1 = s_w;
    float* const sw2 = sw1 + NW1;
    float* const sw3 = sw2 + NW23;
    float* const sw4 = sw3 + NW23;
    for (int k = tid; k < NW1; k += 1024) sw1[k] = w1[k];
    for (int k = tid; k < NW23; k += 1024) {
        sw2[k] = w2[k];
        sw3[k] = w3[k];
    }
    for (int k = tid; k < NW4; k += 1024) sw4[k] = w4[k];
    __syncthreads();
    // channel c = 0 .. 97: layer c / 32 (layer 4: c = 96, 97), output channel c % 32
    for (int c = wave; c < 3 * C + 2; c += 16) {
        const int l = c < 3 * C ? c / C : 3, o = c < 3 * C ? c % C : c - 3 * C;
        const float* w = l == 0 ? sw1 : (l == 1 ? sw2 : (l == 2 ? sw3 : sw4));
        const int per = (l == 0 ? 2 : C) * 9;
        float mx = 0.f, sm = 0.f;
        for (int k = lane; k < per; k += 64) {
            const float a = fabsf(w[o * per + k]);
            mx = fmaxf(mx, a);
            sm += a;
        }
        for (int off = 32; off > 0; off >>= 1) {
            mx = fmaxf(mx, __shfl_xor(mx, off));
            sm += __shfl_xor(sm, off);
        }
        if (lane == 0) {
            s_scale[l][o] = pow2_at_least(mx / 448.f);
            if (l < 3) s_rsum[l][o] = sm;
        }
    }
    __syncthreads();
    if (wave == 0) {
        const float margin = 1.25f;  // covers the rounding of operands (at most 2^-4 each)
        const int o = lane & (C - 1);
        const float bl[3] = { b1[o], b2[o], b3[o] };
        float A = __uint_as_float(s->vmax_bits);
        float s_in = pow2_at_least(A / 448.f);
        if (lane == 0) s->s_v = s_in;
        for (int l = 0; l < 3; ++l) {
            float P = margin * s_rsum[l][o] * A + fabsf(bl[l]);
            for (int off = 16; off > 0; off >>= 1) P = fmaxf(P, __shfl_xor(P, off));
            const float s_out = pow2_at_least(P / 448.f);
            if (lane < C) {
                const float sc = s_scale[l][o] * s_in;
                s->s_w[l][o] = s_scale[l][o];
                s->init[l][o] = bl[l] / sc;
                s->fac[l][o] = sc / s_out;
            }
            if (lane == 0) s->s_a[l] = s_out;
            A = P;
            s_in = s_out;
        }
        if (lane < 2) {
            s->s_w[3][lane] = s_scale[3][lane];
            s->out4[lane] = s_scale[3][lane] * s_in;
        }
    }
    for (int e = tid; e < PACKED; e += 1024) {
        const int l = e & 63, i = l & 15, q = l >> 4;
        float v[8];
        if (e < P1) {
            const int o = (e >> 6) * 16 + i;
            const float r = 1.f / s_scale[0][o];
            for (int j = 0; j < 8; ++j) {
                const int k = 8 * q + j;
                v[j] = k < 18 ? sw1[(o * 2 + (k & 1)) * 9 + (k >> 1)] * r : 0.f;
            }
        } else if (e < P1 + 2 * P2) {
            const int f = e - P1;
            const int layer = f < P2 ? 1 : 2;
            const float* w = f < P2 ? sw2 : sw3;
            const int g = f % P2, t = g / 128, o = ((g >> 6) & 1) * 16 + i;
            const float r = 1.f / s_scale[layer][o];
            for (int j = 0; j < 8; ++j) v[j] = w[(o * C + chan_at(8 * q + j)) * 9 + t] * r;
        } else {
            int o, tap;
            const bool used = conv4_row(16 * ((e - P1 - 2 * P2) >> 6) + i, o, tap);
            const float r = 1.f / s_scale[3][o];
            for (int j = 0; j < 8; ++j) v[j] = used ? sw4[(o * C + chan_at(8 * q + j)) * 9 + tap] * r : 0.f;
        }
        uint64_t word = 0;
        for (int j = 0; j < 8; j += 2) word |= (uint64_t)to_e4m3_pair(v[j], v[j + 1]) << (8 * j);
        packed[e] = (fp8x8)word;
    }
}

struct Fp8 {
    using Op = fp8x8;
    static constexpr int BYTES = 32;
    struct Args {
        const Fp8Scales* sc;
        const float* b4;
    };
    v4f start[2][2], fac[2][2];
    float rv, out4, bo, sum0;

    __device__ __forceinline__ Fp8(const Args& a, bool first, int q, int o)
        : rv(1.f / a.sc->s_v), out4(a.sc->out4[o]), bo(a.b4[o]), sum0(0.f)
    {
#pragma unroll
        for (int l = 0; l < 2; ++l) {
            const int layer = l == 0 ? 0 : first ? 1 : 2;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                start[l][k >> 2][k & 3] = a.sc->init[layer][16 * (k >> 2) + 4 * q + (k & 3)];
                fac[l][k >> 2][k & 3] = a.sc->fac[layer][16 * (k >> 2) + 4 * q + (k & 3)];
            }
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
    k_fp8_clear<<<1, 64, 0, stream>>>(sc);
    const unsigned rb = (unsigned)std::min<int64_t>(512, std::max<int64_t>(1, (count + kMaxThreads - 1) / kMaxThreads));
    k_fp8_absmax<<<rb, kMaxThreads, 0, stream>>>(count, vel, sc);
    k_fp8_prep<<<1, 1024, 0, stream>>>(w.w[0], w.w[1], w.w[2], w.w[3], w.b[0], w.b[1], w.b[2], sc, packed);
    const Plan plan = strip_rows(G, (int)grid);
    k_cnn_fp8<<<(plan.blocks + 7) / 8 * 8, kThreads, 0, stream>>>(G, plan, vel, packed, Fp8::Args{ sc, w.b[3] }, disp);
    hip_check(hipGetLastError(), "fp8 cnn launch");
}

}  // namespace cnnsns
