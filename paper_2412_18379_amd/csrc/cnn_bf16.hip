// Displacement CNN in BF16 on the matrix cores, all four layers fused.
//
// Same network as the FP32 path (3x3 convolutions 2 -> 32 -> 32 -> 32 -> 2,
// zero "same" padding, ReLU between layers, the CNN of Sec. 2.3 in its
// displacement form), computed with BF16 operands (inputs, weights and the
// activations between layers, rounded to nearest even) and FP32
// accumulation; the output displacement is FP32.
//
//
// The pass is the pipeline of cnn_strips.h on v_mfma_f32_16x16x32_bf16.  Biases enter as the accumulators' initial
// values, and ReLU acts on the rounded BF16 pair (rounding to nearest keeps the sign, so the order of the two does not
// change the result).
#include "cnn_strips.h"
#include "common.h"

namespace cnnsns {
namespace {

using namespace strips;

typedef __bf16 bf16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short s16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

__global__ void k_pack_bf16(const float* __restrict__ w1, const float* __restrict__ w2, const float* __restrict__ w3,
                            const float* __restrict__ w4, bf16x8* __restrict__ out)
{
    int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= PACKED) return;
    const int l = e & 63, i = l & 15, q = l >> 4;
    bf16x8 v;
    if (e < P1) {
        const int nb = e >> 6;
        for (int j = 0; j < 8; ++j) {
            const int k = 8 * q + j;
            v[j] = (bf16)(k < 18 ? w1[((nb * 16 + i) * 2 + (k & 1)) * 9 + (k >> 1)] : 0.f);
        }
    } else if (e < P1 + 2 * P2) {
        const int f = e - P1;
        const float* w = f < P2 ? w2 : w3;
        const int g = f % P2, t = g / 128, nb = (g >> 6) & 1;
        for (int j = 0; j < 8; ++j) v[j] = (bf16)w[((nb * 16 + i) * C + chan_at(8 * q + j)) * 9 + t];
    } else {
        int o, tap;
        const bool used = conv4_row(16 * ((e - P1 - 2 * P2) >> 6) + i, o, tap);
        for (int j = 0; j < 8; ++j) v[j] = (bf16)(used ? w4[(o * C + chan_at(8 * q + j)) * 9 + tap] : 0.f);
    }
    out[e] = v;
}

__device__ __forceinline__ uint32_t pair(float v0, float v1)
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{ v0, v1 }, bf16x2));
}

// Channels (i, 16 + i) of one pixel as a packed BF16 pair after ReLU: the
// pair is rounded to nearest even, then every half whose sign bit is set
// (negative, or -0) becomes +0, which is the integer maximum of the bit
// pattern with 0.  The result is ReLU of the rounded value, which equals the
// rounded ReLU.
__device__ __forceinline__ uint32_t relu_pair(float v0, float v1)
{
    const s16x2 r = __builtin_elementwise_max(__builtin_bit_cast(s16x2, pair(v0, v1)), s16x2{ 0, 0 });
    return __builtin_bit_cast(uint32_t, r);
}

struct Bf16 {
    using Op = bf16x8;
    static constexpr int BYTES = 64;
    struct Args {
        const float *b1, *b2, *b3, *b4;
    };
    v4f start[2][2];
    float sum0;

    __device__ __forceinline__ Bf16(const Args& a, bool first, int q, int o) : sum0(a.b4[o])
    {
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            start[0][k >> 2][k & 3] = a.b1[16 * (k >> 2) + 4 * q + (k & 3)];
            start[1][k >> 2][k & 3] = (first ? a.b2 : a.b3)[16 * (k >> 2) + 4 * q + (k & 3)];
        }
    }
    // The LDS serves a 16-byte read in groups of 16 lanes over 64 four-byte banks, a group joining lanes 0-7 with
    // 56-63 (8-15 with 48-55, ...): eight consecutive pixels at chunk q and the next eight at chunk 3 - q, which this
    // puts on distinct banks; and it puts the eight pixels that a store takes at a time on distinct banks of 32.
    static __device__ __forceinline__ int place(int p) { return (p >> 1) & 3; }
    static __device__ __forceinline__ v4f mfma(const Op& a, const Op& b, const v4f& c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
    }
    __device__ __forceinline__ uint32_t vel(float u, float v) const { return pair(u, v); }
    static __device__ __forceinline__ Op gather(const uint32_t (&v)[4])
    {
        Op x;
        __builtin_memcpy(&x, v, sizeof x);
        return x;
    }
    template <int LAYER>
    __device__ __forceinline__ void act(const v4f& lo, const v4f& hi, uint32_t (&w)[4]) const
    {
#pragma unroll
        for (int r = 0; r < 4; ++r) w[r] = relu_pair(lo[r], hi[r]);
    }
    __device__ __forceinline__ float sum(float s) const { return s; }
};

__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_cnn_bf16(
    int32_t G, Plan plan, const float* __restrict__ vel, const bf16x8* __restrict__ packed, Bf16::Args b,
    float* __restrict__ disp)
{
    pass<Bf16>(G, plan, vel, packed, b, disp);
}

}  // namespace

size_t cnn_bf16_workspace_bytes()
{
    return sizeof(bf16x8) * (size_t)PACKED;
}

void cnn_bf16_pack(const cnnsns_cnn& w, void* packed, hipStream_t stream)
{
    k_pack_bf16<<<(PACKED + 255) / 256, 256, 0, stream>>>(w.w[0], w.w[1], w.w[2], w.w[3],
                                                      static_cast<bf16x8*>(packed));
    hip_check(hipGetLastError(), "bf16 weight packing");
}

void cnn_bf16_forward(int32_t G, const float* vel, const void* packed, const cnnsns_cnn& w, float* disp,
                      unsigned grid, hipStream_t stream)
{
    const Plan plan = strip_rows(G, (int)grid);
    k_cnn_bf16<<<(plan.blocks + 7) / 8 * 8, kThreads, 0, stream>>>(
        G, plan, vel, static_cast<const bf16x8*>(packed), Bf16::Args{ w.b[0], w.b[1], w.b[2], w.b[3] }, disp);
    hip_check(hipGetLastError(), "bf16 cnn launch");
}

}  // namespace cnnsns
