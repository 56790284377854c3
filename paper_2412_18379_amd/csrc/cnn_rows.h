// The FP32 forward pass of the 2D displacement CNN (cnn.hip) as two kernels that stream rows, for all but
// mid-sized overlays.
//
// k_rows12_f32 runs conv1 and conv2, k_rows34_f32 conv3 and conv4, with the 32-channel activation
// between them in memory, pixel-major ([G][G][32]).  A block owns a strip of
// 256 columns and a segment of rows, and walks down it one row per step; each
// of its eight wavefronts owns 32 columns.  A step takes one input row of the
// 32 -> 32 layer from LDS (double-buffered: the next row is being written by
// conv1, or by loads from memory, meanwhile), transforms and splits it once,
// and adds its products to the three output rows it feeds, whose accumulators
// stay in registers; the oldest of them is then complete.  So no row is
// computed twice inside a segment and there is one barrier per row.
//
// The 32 -> 32 layers use the minimal filtering algorithm F(2,3) along the row
// (Winograd; Lavin and Gray, 2016): for two output columns and one row of the
// filter, four products replace six,
//   Y = A^T [ (G g) (.) (B^T d) ],   d four input columns, g three taps,
//   B^T d = (d0 - d2, d1 + d2, d2 - d1, d1 - d3),
//   G g   = (g0, (g0 + g1 + g2)/2, (g0 - g1 + g2)/2, g2),
//   Y     = (m0 + m1 + m2, m1 - m2 - m3).
// Summed over the 32 input channels each of the 4 x 3 products (position,
// filter row) is a channel contraction, and runs as six BF16 matrix
// instructions on operands split into three BF16 values each (split.h), with
// FP32's precision.
//
// What bounds it (G = 4096): a wavefront's row is 164 matrix instructions (168 in the second kernel; 16.5 cycles each)
// and about 600 vector instructions (690; 3 cycles), and on one SIMD the two add up: two wavefronts that mix them
// take 14 + 3 n cycles per matrix instruction with n vector instructions, measured.  That sum is three quarters of
// the pass, 2.50 ms in repeated calls.  The other splits of the work: the tile form (FP32 matrix instruction,
// F(2x2, 3x3), cnn.hip) 3.67 ms; direct convolution on operands split where they enter LDS (216 matrix
// instructions a row, 400 vector ones) 3.03, when this form took 2.67.  F(2x2, 3x3) on split operands has the same sum as
// F(2,3): a third fewer matrix instructions, but it splits four transformed values per input instead of two,
// and its 96 KiB of weights do not fit in LDS beside two rows of 258 pixels.
#pragma once

#include "common.h"
#include "lds_copy.h"
#include "split.h"

namespace cnnsns {
namespace rows {

constexpr int C = 32;                     // hidden channels
constexpr int SW = 256;                   // columns of a strip
constexpr int kWaves = 8;                 // wavefronts of a block, two per SIMD
constexpr int kThreads = 64 * kWaves;
constexpr int WC = SW / kWaves;           // columns of a wavefront: sixteen pairs, one matrix block
static_assert(WC == 32, "a wavefront's columns are the 16 column pairs of one matrix block");
constexpr int NF32 = 4 * 3 * 2 * 3;       // weight operands of a 32 -> 32 layer: position, filter row, half, part
constexpr int NU = NF32 * 64;             // bf16x8 per layer (72 KiB)
constexpr int NF1 = 5 * 2;                // conv1: five K steps, two halves of the output channels
constexpr int NF4 = 2 * 3;                // conv4: output component, part
constexpr int ROWP = SW / 2 + 1;          // pixel pairs of a row in LDS (the strip and one column each side)
constexpr int ROWV = ROWP * 16;           // v4f of it
constexpr int VPX = SW + 4;               // velocity pixels of a row (two columns each side)

// Prepared operands at the start of the workspace.
constexpr size_t kOffU2 = 0, kOffU3 = kOffU2 + NU * sizeof(bf16x8), kOffW1 = kOffU3 + NU * sizeof(bf16x8),
                 kOffW4 = kOffW1 + NF1 * 64 * sizeof(bf16x8), kOffZero = kOffW4 + NF4 * 64 * sizeof(bf16x8),
                 kOffEdge = kOffZero + 256;

// Bytes of the partial sums that neighbouring strips exchange (k_strip_edges).
inline size_t edge_bytes(int32_t G)
{
    const size_t n = (size_t)((G + SW - 1) / SW - 1) * 2 * (size_t)G * 2 * sizeof(float);
    return (n + 255) / 256 * 256;
}

// A row of 32-channel pixels in LDS: 16-byte chunks (four channels), a pixel pair k = 256 bytes.  Chunk
// c of pixel 2k + p is slot (8p + c + 2k) mod 16 of its pair.  The LDS serves a 16-byte read in groups
// of 16 lanes over 64 four-byte banks, a group joining lanes 0-7 with 56-63 (8-15 with 48-55, ...): here
// eight consecutive pairs at one chunk and the next eight at another, at the same p.  The rotation by 2k
// puts each eight on the slots of one parity, so the sixteen are distinct when the two chunks differ in
// parity, which chunk_of arranges.
__device__ __forceinline__ int row_slot(int pair, int p, int c)
{
    return pair * 16 + ((8 * p + c + 2 * pair) & 15);
}

// The chunk that lane group q reads as the first (h = 0) or second (h = 1) half of its eight input
// channels: 2q and 2q + 1, in the other order for q = 2, 3.
__host__ __device__ constexpr int chunk_of(int q, int h)
{
    return 2 * q + (h ^ (q >> 1));
}

// Weight operands of all four layers, in one launch (they depend on the call's weights; BF16 parts of
// values formed in FP64), and a run of zeros.
//   32 -> 32: u[((((pos * 3 + dy) * 2 + nb) * 3 + part) * 64 + l)][j] = part of (G g)[pos] for output channel
//     16 nb + l%16, input channel 4 chunk_of(l/16, j/4) + j%4 and filter row dy: the A operand
//     (row = output channel, k = input channel) in the channel order in which lanes read a row.
//   conv1: w1[(st * 2 + nb) * 64 + l]: lane group q of step st takes slot t = 4 st + q.  Slots 0..8 are the
//     taps against a pixel's record (u_h, v_h, u_m, v_m, u_l, v_l, u_h, v_h) with weights
//     (w_h, w_h, w_h, w_h, w_h, w_h, w_m, w_m), slots 9..17 the taps again with (w_l, w_l, w_m, w_m, 0...):
//     together the six products.
//   conv4: w4[(o * 3 + part) * 64 + l]: row 4 dx + dy = filter tap (dy, dx) of output component o (rows
//     with dy = 3 or dx = 3 zero), k = the channel the 32 -> 32 layer's result leaves in that place:
//     lane group q, element j holds channel 16 (j/4) + 4 q + j%4.
static __global__ void k_rows_prep(const float* __restrict__ w1, const float* __restrict__ w2, const float* __restrict__ w3,
                           const float* __restrict__ w4, char* __restrict__ ws)
{
    int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < 2 * NU) {
        const int layer = k / NU;
        k -= layer * NU;
        const int l = k & 63, part = (k >> 6) % 3, nb = (k / 192) & 1, dy = (k / 384) % 3, pos = k / 1152;
        const float* w = layer ? w3 : w2;
        bf16x8 v;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float* g = w + ((16 * nb + (l & 15)) * C + 4 * chunk_of(l >> 4, j >> 2) + (j & 3)) * 9 + 3 * dy;
            const double g0 = g[0], g1 = g[1], g2 = g[2];
            const double u = pos == 0 ? g0 : pos == 1 ? 0.5 * (g0 + g1 + g2) : pos == 2 ? 0.5 * (g0 - g1 + g2) : g2;
            v[j] = split_part(u, part);
        }
        reinterpret_cast<bf16x8*>(ws + (layer ? kOffU3 : kOffU2))[k] = v;
        return;
    }
    k -= 2 * NU;
    if (k < NF1 * 64) {
        const int l = k & 63, nb = (k >> 6) & 1, st = k >> 7, o = 16 * nb + (l & 15), t = 4 * st + (l >> 4);
        bf16x8 v;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            double x = 0.0;
            int part = 0;
            if (t < 9) {
                x = w1[(o * 2 + (j & 1)) * 9 + t];
                part = j < 6 ? 0 : 1;
            } else if (t < 18 && j < 4) {
                x = w1[(o * 2 + (j & 1)) * 9 + t - 9];
                part = j < 2 ? 2 : 1;
            }
            v[j] = split_part(x, part);
        }
        reinterpret_cast<bf16x8*>(ws + kOffW1)[k] = v;
        return;
    }
    k -= NF1 * 64;
    if (k < NF4 * 64) {
        const int l = k & 63, part = (k >> 6) % 3, o = k / 192, row = l & 15, dx = row >> 2, dy = row & 3;
        bf16x8 v;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int ch = 16 * (j >> 2) + 4 * (l >> 4) + (j & 3);
            v[j] = split_part(dx < 3 && dy < 3 ? (double)w4[(o * C + ch) * 9 + 3 * dy + dx] : 0.0, part);
        }
        reinterpret_cast<bf16x8*>(ws + kOffW4)[k] = v;
        return;
    }
    k -= NF4 * 64;
    if (k < 16) reinterpret_cast<v4f*>(ws + kOffZero)[k] = v4f{ 0.f, 0.f, 0.f, 0.f };
}
constexpr int kRowsPrepItems = 2 * NU + (NF1 + NF4) * 64 + 16;

// Accumulators of one output row of a wavefront: a[pos][nb], lane (i, q): channels 16 nb + 4q + r of pair i.
typedef v4f Acc[4][2];

// The 32 -> 32 layer of one wavefront, row by row.  A row's work is twelve stages (position, filter row) of
// twelve matrix instructions, in three parts of four: the two halves of the output channels take turns, so
// that an instruction does not wait for the one before it (a dependent one issues 35 cycles later, twice
// an instruction's 16).  The compiled order is pinned (sched_barrier): a part's issue is shared with the LDS
// reads of weights used two parts on, the splitting of the next position's input, the addition of the previous
// stage's small products and a slice of the step's other work, which the compiler would otherwise put
// between the stages.  The last position's stages are left for the next step, after the barrier: they keep
// the matrix cores busy while the new row is read and its first position split.
constexpr int kStages = 12, kTail = 9;  // stages of a row; those from kTail on run in the next step
struct RowConv {
    const bf16x8* u;                      // the layer's weights in LDS, at the lane
    const v4f* bias;                      // and its biases, then their negatives, at the lane
    bf16x8 wh[2][2], wm[2], wl[2];        // [stage parity][half], [half]
    v4f s[2][2];                          // small products of this stage and the previous one
    v4f d[4][2];                          // the row's four input columns of the lane's pair, eight channels
    u32x4 v[2][3];                        // parts of this and the next position's transformed input

    __device__ __forceinline__ void load_weights(bf16x8 (&w)[2], int st, int part)
    {
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) w[nb] = u[((st * 2 + nb) * 3 + part) * 64];
    }
    // before the first row: its weights, and nothing left of a row before it
    __device__ __forceinline__ void start()
    {
        load_weights(wh[kTail & 1], kTail, 0);
        load_weights(wl, kTail, 2);
#pragma unroll
        for (int part = 0; part < 3; ++part) v[1][part] = u32x4{ 0, 0, 0, 0 };
    }
    // input columns of the row (pairs 16 wave .. of `row`, whose pixel 0 is the column before the strip)
    __device__ __forceinline__ void load_row(const v4f* __restrict__ row, int wave, int lane)
    {
        asm volatile("" : "+v"(lane));  // the addresses are formed per row, not held in registers
#pragma unroll
        for (int col = 0; col < 4; ++col)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                d[col][h] = row[row_slot(16 * wave + (lane & 15) + (col >> 1), col & 1, chunk_of(lane >> 4, h))];
    }
    // channel pair k of position pos: transform and split
    __device__ __forceinline__ void split(int pos, int k)
    {
        float x[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int h = k >> 1, c = 2 * (k & 1) + j;
            x[j] = pos == 0 ? d[0][h][c] - d[2][h][c] : pos == 1 ? d[1][h][c] + d[2][h][c]
                 : pos == 2 ? d[2][h][c] - d[1][h][c] : d[1][h][c] - d[3][h][c];
        }
        uint32_t h, m, l;
        split_pair(x[0], x[1], h, m, l);
        v[pos & 1][0][k] = h;
        v[pos & 1][1][k] = m;
        v[pos & 1][2][k] = l;
    }
    // What the products of position pos are added to in a fresh row: the bias of the layer enters output
    // column 0 through m0 and column 1 through -m3.
    __device__ __forceinline__ v4f origin(int pos, int nb) const
    {
        return pos == 0 ? bias[4 * nb] : pos == 3 ? bias[8 + 4 * nb] : v4f{ 0.f, 0.f, 0.f, 0.f };
    }
    // part `sub` of stage st's products into acc (fresh: a new row)
    __device__ __forceinline__ void products(int st, int sub, bool fresh, v4f (&acc)[2])
    {
        const v4f zero = v4f{ 0.f, 0.f, 0.f, 0.f };
        const int p = st / 3 & 1;
        const bf16x8 vh = __builtin_bit_cast(bf16x8, v[p][0]), vm = __builtin_bit_cast(bf16x8, v[p][1]),
                     vl = __builtin_bit_cast(bf16x8, v[p][2]);
        v4f(&t)[2] = s[st & 1];
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
            t[nb] = sub == 0 ? mfma_bf16(wl[nb], vh, zero)
                  : sub == 1 ? mfma_bf16(wh[st & 1][nb], vl, t[nb]) : mfma_bf16(wm[nb], vm, t[nb]);
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) {
            if (sub == 0)
                acc[nb] = mfma_bf16(wh[st & 1][nb], vh, fresh ? origin(st / 3, nb) : acc[nb]);
            else
                t[nb] = sub == 1 ? mfma_bf16(wh[st & 1][nb], vm, t[nb]) : mfma_bf16(wm[nb], vh, t[nb]);
        }
    }
    // Stages [B, E) of a row: c0 (a new row) takes filter row 0, c1 row 1, c2 row 2.  While position p runs,
    // position p + 1 is split (after position 3: position 0 of the row in d).
    template <int B, int E>
    __device__ __forceinline__ void stages(Acc& c0, Acc& c1, Acc& c2)
    {
        auto acc_of = [&](int st) -> v4f(&)[2] { return (st % 3 == 0 ? c0 : st % 3 == 1 ? c1 : c2)[st / 3]; };
        auto add_small = [&](int st) {
            acc_of(st)[0] += s[st & 1][0];
            acc_of(st)[1] += s[st & 1][1];
        };
#pragma unroll
        for (int st = B; st < E; ++st) {
            const int dy = st % 3, next = (st + 1) % kStages;
#pragma unroll
            for (int sub = 0; sub < 3; ++sub) {
                __builtin_amdgcn_sched_barrier(0);
                if (sub == 0) load_weights(wm, st, 1);
                if (sub == 1) load_weights(wh[next & 1], next, 0);
                if (sub == 2) load_weights(wl, next, 2);
                products(st, sub, dy == 0, acc_of(st));
                if (sub == 0 && st > B) add_small(st - 1);
                if (dy > 0 && sub > 0) split((st / 3 + 1) & 3, 2 * (dy - 1) + sub - 1);
                // the reads first, then the products with the part's other work between them
                __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        add_small(E - 1);
    }
};

// The two output columns of every pair: y[e][nb], channels 16 nb + 4q + r of column 2i + e.
__device__ __forceinline__ void wino_out(const Acc& m, v4f (&y)[2][2])
{
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
        y[0][nb] = m[0][nb] + m[1][nb] + m[2][nb];
        y[1][nb] = m[1][nb] - m[2][nb] - m[3][nb];
    }
}

// x summed over the four lanes l % 16 + 16 k of its 16-lane column: x + (x of lane l ^ 16), then the
// same with lane l ^ 32, through the lane-swap instructions (no trip through the LDS).  With both
// operands x, the swap returns x of lane l in one half and of its partner in the other, so their sum
// is x_l + x_(l ^ 16); the two addends may come in either order, which leaves the sum unchanged.
__device__ __forceinline__ float sum_lane_column(float x)
{
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// x of the lane one to the left (right) in the 16-lane column row, 0 past its end.
__device__ __forceinline__ float from_left(float x)
{
    return __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x111, 0xf, 0xf, true));  // row_shr:1
}
__device__ __forceinline__ float from_right(float x)
{
    return __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x101, 0xf, 0xf, true));  // row_shl:1
}

// Row segments of the strips: a launch is one round of blocks, one per compute unit (the LDS footprint allows
// one).  The last strip, which may be narrow, has segments of its own length.
struct RowPlan {
    int strips, segs, seg_rows;  // segments of a full strip
    int last_segs, last_rows;    // of the last strip
    __host__ __device__ int blocks() const { return (strips - 1) * segs + last_segs; }
    // strip and rows [r0, r1) of block s < blocks()
    __host__ __device__ void at(int s, int G, int& strip, int& r0, int& r1) const
    {
        const bool last = s >= (strips - 1) * segs;
        strip = last ? strips - 1 : s / segs;
        r0 = (s - strip * segs) * (last ? last_rows : seg_rows);
        r1 = r0 + (last ? last_rows : seg_rows);
        r1 = r1 < G ? r1 : G;
    }
};

// The plan with the smallest longest block.  A block's time is its rows and what it spends besides them (its
// weights, halo rows: about three rows' worth); a strip of at most half the wavefronts, one per SIMD, takes
// 0.62 of a full one's time a row (14 us for one row against 39 for four at the two widths).
inline RowPlan row_plan(int G, int cus)
{
    auto cdiv = [](int a, int b) { return (a + b - 1) / b; };
    RowPlan best{};
    best.strips = cdiv(G, SW);
    const int full = best.strips - 1, lastw = G - full * SW;
    const double t = lastw <= SW / 2 ? 0.62 : 1.0;
    double cost = -1.0;
    for (int nl = 1; nl <= (cus > best.strips ? cus - full : 1); ++nl) {
        const int nf = full ? (cus - nl > full ? (cus - nl) / full : 1) : 1;
        const int rf = cdiv(G, nf), rl = cdiv(G, nl);
        const double c = t * (rl + 3), cf = full ? rf + 3.0 : 0.0, worst = c > cf ? c : cf;
        if (cost < 0.0 || worst < cost) {
            cost = worst;
            best.seg_rows = rf;
            best.segs = cdiv(G, rf);
            best.last_rows = rl;
            best.last_segs = cdiv(G, rl);
        }
    }
    return best;
}

// Segments are handed out in runs per XCD (workgroups go to the 8 XCDs round-robin by id), so that those that
// share halo rows meet in one L2.  False past the last segment.
__device__ __forceinline__ bool block_segment(int G, const RowPlan& p, int& x0, int& r0, int& r1)
{
    const int per = gridDim.x / 8, s = (blockIdx.x % 8) * per + blockIdx.x / 8;
    if (s >= p.blocks()) return false;
    int strip;
    p.at(s, G, strip, r0, r1);
    x0 = strip * SW;
    return true;
}

// The layer's weights, straight into LDS; the caller waits (lds_copies_arrived).
__device__ __forceinline__ void load_u(const bf16x8* __restrict__ u, bf16x8* __restrict__ s_u, int wave, int lane)
{
    static_assert(NU % kThreads == 0, "whole rounds");
#pragma unroll
    for (int k = 0; k < NU / kThreads; ++k) {
        const int at = k * kThreads + wave * 64;
        lds_copy16(u + at + lane, s_u + at);
    }
}

// conv1 + ReLU then conv2 + ReLU -> act2 [G][G][32].  What bounds it: matrix instructions, 288 of
// conv2's and 42 of conv1's per SIMD and row of 256 columns (16 cycles each).
static __global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_rows12_f32(
    int32_t G, RowPlan plan, const float* __restrict__ vel, const char* __restrict__ ws,
    const float* __restrict__ b1, const float* __restrict__ b2, float* __restrict__ act2)
{
    __shared__ bf16x8 s_u[NU];
    __shared__ v4f s_row[2][ROWV];                      // conv1's output rows a (in use) and a + 1
    __shared__ bf16x8 s_w1[NF1 * 64];
    __shared__ uint32_t s_vel[4][3][VPX];               // (u, v) of rows a .. a + 3 in three BF16 parts
    __shared__ v4f s_b[3][C / 4];                       // biases of conv1, of conv2 and their negatives

    int x0, r0, r1;
    if (!block_segment(G, plan, x0, r0, r1)) return;
    const int tid = threadIdx.x, lane = tid & 63, q = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t GG = (int64_t)G * G;
    const bool active = x0 + WC * wave < G;  // the wavefront has columns inside the grid

    for (int k = tid; k < NF1 * 64; k += kThreads) s_w1[k] = reinterpret_cast<const bf16x8*>(ws + kOffW1)[k];
    if (tid < 3 * C) reinterpret_cast<float*>(s_b)[tid] = tid < C ? b1[tid] : tid < 2 * C ? b2[tid - C] : -b2[tid - 2 * C];

    // velocity row v, column x0 - 2 + tid, loaded unconditionally from a clamped position; what lies
    // outside the grid is zeroed when the parts are written
    float pu = 0.f, pv = 0.f;
    auto fetch_vel = [&](int v) {
        int t = tid;
        asm volatile("" : "+v"(t));  // positions are formed per row, not held in registers
        if (t < VPX) {
            const float* row = vel + (int64_t)min(max(v, 0), G - 1) * G;
            const unsigned at = min(max(x0 - 2 + t, 0), G - 1);
            pu = row[at];
            pv = (row + GG)[at];
        }
    };
    auto stash_vel = [&](int v) {
        int t = tid;
        asm volatile("" : "+v"(t));
        if (t < VPX) {
            const bool in = (unsigned)v < (unsigned)G && (unsigned)(x0 - 2 + t) < (unsigned)G;
            uint32_t h, m, l;
            split_pair_any(in ? pu : 0.f, in ? pv : 0.f, h, m, l);
            s_vel[v & 3][0][t] = h;
            s_vel[v & 3][1][t] = m;
            s_vel[v & 3][2][t] = l;
        }
    };
    // conv1 of row a into its row buffer: 16-pixel blocks wave and wave + 8 of the 258 pixels, and
    // in turn the last two pixels; zero outside the grid (conv2's padding).  Lane group q of step st takes tap
    // (4 st + q) mod 9: column (st + q) mod 3, and of the three velocity rows one of two that the step names (past tap 17,
    // where the weights are zero, any pixel of the window).
    auto conv1 = [&](int a) {
        v4f* dst = s_row[a & 1];
        int ln = lane;
        asm volatile("" : "+v"(ln));  // the addresses are formed per row, not held in registers
        const int i = ln & 15, q = ln >> 4;
        int row[3], col[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) row[k] = ((a + k - 1) & 3) * 3 * VPX;
        col[0] = i + (q == 3 ? 0 : q);
        col[1] = i + (q == 2 ? 0 : q == 3 ? 1 : q + 1);
        col[2] = i + (q == 0 ? 2 : q - 1);
        auto blocks = [&](auto nblk, int mb0) {
            constexpr int NB = decltype(nblk)::value;  // 1: the block of the last two pixels
            v4f acc[NB][2];
#pragma unroll
            for (int u = 0; u < NB; ++u)
#pragma unroll
                for (int nb = 0; nb < 2; ++nb) acc[u][nb] = s_b[0][4 * nb + q];
#pragma unroll
            for (int st = 0; st < 5; ++st) {
                if (st == 3) __builtin_amdgcn_sched_barrier(0);  // not all operands at once: registers
                constexpr int first[5] = { 0, 1, 2, 1, 2 }, other[5] = { 1, 2, 0, 2, 0 }, lanes[5] = { 3, 2, 1, 3, 2 };
                const uint32_t* src = s_vel[0][0] + (q < lanes[st] ? row[first[st]] : row[other[st]]);
#pragma unroll
                for (int u = 0; u < NB; ++u) {
                    const int px = 16 * (mb0 + 8 * u) + col[st % 3];
                    const uint32_t* at = src + (NB == 1 ? min(px, VPX - 1) : px);
                    const uint32_t h = at[0];
                    const bf16x8 b = __builtin_bit_cast(bf16x8, u32x4{ h, at[VPX], at[2 * VPX], h });
#pragma unroll
                    for (int nb = 0; nb < 2; ++nb) acc[u][nb] = mfma_bf16(s_w1[(st * 2 + nb) * 64 + ln], b, acc[u][nb]);
                }
            }
#pragma unroll
            for (int u = 0; u < NB; ++u) {
                const int px = 16 * (mb0 + 8 * u) + i;
                const bool in = (unsigned)(x0 - 1 + px) < (unsigned)G && (unsigned)a < (unsigned)G;
                const float top = in ? __builtin_inff() : 0.f;
                if (NB > 1 || px < SW + 2) {
#pragma unroll
                    for (int nb = 0; nb < 2; ++nb) {
                        v4f v = acc[u][nb];
#pragma unroll
                        for (int r = 0; r < 4; ++r) v[r] = __builtin_amdgcn_fmed3f(v[r], 0.f, top);
                        dst[row_slot(px >> 1, px & 1, 4 * nb + q)] = v;
                    }
                }
            }
        };
        blocks(std::integral_constant<int, 2>{}, wave);
        if (wave == (a & 7)) blocks(std::integral_constant<int, 1>{}, 16);
    };

    // the first four rows' loads together, one wait for memory; conv2's weights land while conv1 runs (the kernels of a
    // pass on 128 x 128 cells: 36.7 us with four waits and the weights before them, 36.2 so)
    float u[4], v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        fetch_vel(r0 - 2 + k);
        u[k] = pu;
        v[k] = pv;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        pu = u[k];
        pv = v[k];
        stash_vel(r0 - 2 + k);
    }
    load_u(reinterpret_cast<const bf16x8*>(ws + kOffU2), s_u, wave, lane);
    __syncthreads();
    conv1(r0 - 1);
    lds_copies_arrived();
    __syncthreads();

    RowConv rc;
    rc.u = s_u + lane;
    rc.bias = s_b[1] + q;
    rc.start();
    // output row y from its accumulators
    auto emit = [&](int y, const Acc& m) {
        v4f o[2][2];
        wino_out(m, o);
        int ln = lane;
        asm volatile("" : "+v"(ln));
        const int i = ln & 15, q = ln >> 4;
        float* out = act2 + (int64_t)y * G * C;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int gx = x0 + WC * wave + 2 * i + e;
            if (gx < G) {
#pragma unroll
                for (int nb = 0; nb < 2; ++nb) {
                    v4f v = o[e][nb];
#pragma unroll
                    for (int r = 0; r < 4; ++r) v[r] = fmaxf(v[r], 0.f);
                    *reinterpret_cast<v4f*>(out + (unsigned)(gx * C + 16 * nb + 4 * q)) = v;
                }
            }
        }
    };
    // Step a: the rest of input row a - 1, whose accumulators are c0, c1, c2, which completes output row
    // a - 2; then input row a into c2 (now fresh), c0, c1.
    auto step = [&](int a, Acc& c0, Acc& c1, Acc& c2) {
        if (a + 3 <= r1 + 1) fetch_vel(a + 3);  // lands while the row computes
        if (active) {
            rc.load_row(s_row[a & 1], wave, lane);
            rc.stages<kTail, kStages>(c0, c1, c2);
            if (a - 2 >= r0) emit(a - 2, c2);
        }
        if (a + 1 <= r1) conv1(a + 1);
        if (a <= r1) {
            if (active) rc.stages<0, kTail>(c2, c0, c1);
            if (a + 3 <= r1 + 1) stash_vel(a + 3);
            __syncthreads();
        }
    };
    Acc c0, c1, c2;
    for (int pos = 0; pos < 4; ++pos)
        for (int nb = 0; nb < 2; ++nb) c0[pos][nb] = c1[pos][nb] = c2[pos][nb] = v4f{ 0.f, 0.f, 0.f, 0.f };
    for (int a = r0 - 1; a <= r1 + 1; a += 3) {
        step(a, c0, c1, c2);
        if (a + 1 <= r1 + 1) step(a + 1, c2, c0, c1);
        if (a + 2 <= r1 + 1) step(a + 2, c1, c2, c0);
    }
}

// conv3 + ReLU then conv4 -> disp.  conv4 takes conv3's result in the registers it lies in: for each
// output component one matrix block with rows (dx, dy), K = the 32 channels, so that a lane holds, for
// its column, one dx and the three dy, which feed three output rows: the running sums move down one
// element per step and the element for dy = 2 completes a row.  The three dx are then summed across the
// four lanes of a column, from the neighbouring columns' lanes; the columns at a wavefront's sides
// get their neighbour's part through LDS one step later, those at a strip's sides through memory
// (k_strip_edges).  What bounds it: matrix instructions, 336 per SIMD and row of 256 columns.
static __global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_rows34_f32(
    int32_t G, RowPlan plan, const float* __restrict__ act2, const char* __restrict__ ws,
    const float* __restrict__ b3, const float* __restrict__ b4, float* __restrict__ edge, float* __restrict__ disp)
{
    __shared__ bf16x8 s_u[NU];
    __shared__ v4f s_row[2][ROWV];                  // act2 rows a (in use) and a + 1 (arriving)
    __shared__ bf16x8 s_w4[NF4 * 64];
    __shared__ float s_side[2][kWaves][4];          // a row's parts for the columns left and right of a wavefront
    __shared__ v4f s_b[2][C / 4];                   // biases of conv3 and their negatives
    // a thread's two columns of the row completed in the previous step, without their sides (lane group q: component q)
    __shared__ float2 s_held[kThreads];
    __shared__ int s_from[4][kThreads];             // a thread's places in a row: float offset, or -1 outside the grid

    int x0, r0, r1;
    if (!block_segment(G, plan, x0, r0, r1)) return;
    const int tid = threadIdx.x, lane = tid & 63, i = lane & 15, q = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t GG = (int64_t)G * G;
    const bool active = x0 + WC * wave < G;
    const int strip = x0 / SW, strips = (G + SW - 1) / SW;

    // act2 row a straight into its LDS buffer, 16 bytes a lane: a lane's place in LDS is given by its
    // position, so it picks the pixel and chunk that row_slot puts there; zeros outside the grid
    // (conv3's padding).  Its pixels are the same in every row: looked up, not formed again (16 instructions each).
    auto place = [&](int k) {
        const int pair = k >> 4, pc = (k - 2 * pair) & 15, gx = x0 - 1 + 2 * pair + (pc >> 3);
        return (unsigned)gx < (unsigned)G ? gx * C + 4 * (pc & 7) : -1;
    };
#pragma unroll
    for (int u = 0; u < 4; ++u) s_from[u][tid] = place((wave + kWaves * u) * 64 + lane);  // read by this thread only
    auto load_row = [&](int a) {
        const float* src = act2 + (int64_t)a * G * C;
        const float* zero = reinterpret_cast<const float*>(ws + kOffZero);
        const bool row_in = (unsigned)a < (unsigned)G;
        auto piece = [&](int p0, int from) { lds_copy16(row_in && from >= 0 ? src + (unsigned)from : zero, s_row[a & 1] + p0 * 64); };
        static_assert((ROWV + 63) / 64 == 4 * kWaves + 1, "four pieces per wavefront and one in turn");
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            int ln = lane;
            asm volatile("" : "+v"(ln));  // not all places at once: registers
            piece(wave + kWaves * u, s_from[u][64 * wave + ln]);
        }
        if (wave == (a & 7)) {
            int ln = lane;
            asm volatile("" : "+v"(ln));
            if (4 * kWaves * 64 + ln < ROWV) piece(4 * kWaves, place(4 * kWaves * 64 + ln));
        }
    };

    load_row(r0 - 2);
    load_u(reinterpret_cast<const bf16x8*>(ws + kOffU3), s_u, wave, lane);
    for (int k = tid; k < NF4 * 64; k += kThreads) s_w4[k] = reinterpret_cast<const bf16x8*>(ws + kOffW4)[k];
    if (tid < 2 * C) reinterpret_cast<float*>(s_b)[tid] = tid < C ? b3[tid] : -b3[tid - C];
    if (tid < 2 * kWaves * 4) (&s_side[0][0][0])[tid] = 0.f;  // wavefronts past the grid leave theirs at zero
    const float bias4[2] = { b4[0], b4[1] };
    lds_copies_arrived();
    __syncthreads();

    v4f part[2][2];      // [column e][component o]: running sums for three output rows
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int o = 0; o < 2; ++o) part[e][o] = v4f{ 0.f, 0.f, 0.f, 0.f };

    // writes output row yo from `held` and the neighbouring wavefronts' parts of it: lane group q < 2 component q
    auto finish = [&](int yo) {
        int ln = lane;
        asm volatile("" : "+v"(ln));
        const int i = ln & 15, q = ln >> 4;
        const float left = s_side[yo & 1][wave > 0 ? wave - 1 : 0][2 + (q & 1)];
        const float right = s_side[yo & 1][wave + 1 < kWaves ? wave + 1 : kWaves - 1][q & 1];
        const unsigned gx = x0 + WC * wave + 2 * i;
        const float2 held = s_held[64 * wave + ln];
        const float d0 = i == 0 && wave > 0 ? held.x + left : held.x;
        const float d1 = i == 15 && wave + 1 < kWaves ? held.y + right : held.y;
        float* to = disp + (int64_t)yo * G + gx;
        if (q == 1) to += GG;
        if (q < 2 && gx + 1 < (unsigned)G) {
            to[0] = d0;
            to[1] = d1;
        } else if (q < 2 && gx < (unsigned)G) {
            to[0] = d0;
        }
    };
    RowConv rc;
    rc.u = s_u + lane;
    rc.bias = s_b[0] + q;
    rc.start();
    // Step a: the rest of input row a - 1 (accumulators c0, c1, c2), which completes conv3's row a - 2 and
    // with it conv4's row a - 3; then input row a into c2 (now fresh), c0, c1.
    auto step = [&](int a, Acc& c0, Acc& c1, Acc& c2) {
        if (a + 1 <= r1 + 1) load_row(a + 1);  // lands while the row computes
        if (active) {
            rc.load_row(s_row[a & 1], wave, lane);
            if (a - 4 >= r0) finish(a - 4);
            rc.stages<kTail, kStages>(c0, c1, c2);
            if (a - 1 >= r0) {
                const int y3 = a - 2;  // the row of conv3 that is complete
#pragma unroll
                for (int e = 0; e < 2; ++e)
#pragma unroll
                    for (int o = 0; o < 2; ++o) part[e][o] = v4f{ 0.f, part[e][o][0], part[e][o][1], 0.f };
                if ((unsigned)y3 < (unsigned)G) {  // rows outside the grid are conv4's zero padding
                    v4f y[2][2];
                    wino_out(c2, y);
                    Split8 v[2];
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        // columns outside the grid are conv4's zero padding
                        const float top = x0 + WC * wave + 2 * i + e < G ? __builtin_inff() : 0.f;
#pragma unroll
                        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
                            for (int r = 0; r < 4; ++r) y[e][nb][r] = __builtin_amdgcn_fmed3f(y[e][nb][r], 0.f, top);
                        v[e] = split8(y[e][0], y[e][1]);
                    }
#pragma unroll
                    for (int o = 0; o < 2; ++o) {
                        const bf16x8 wh = s_w4[(o * 3 + 0) * 64 + lane], wm = s_w4[(o * 3 + 1) * 64 + lane],
                                     wl = s_w4[(o * 3 + 2) * 64 + lane];
                        v4f s[2];
#pragma unroll
                        for (int e = 0; e < 2; ++e) s[e] = mfma_bf16(wl, v[e].h, v4f{ 0.f, 0.f, 0.f, 0.f });
#pragma unroll
                        for (int e = 0; e < 2; ++e) s[e] = mfma_bf16(wh, v[e].l, s[e]);
#pragma unroll
                        for (int e = 0; e < 2; ++e) s[e] = mfma_bf16(wm, v[e].m, s[e]);
#pragma unroll
                        for (int e = 0; e < 2; ++e) s[e] = mfma_bf16(wm, v[e].h, s[e]);
#pragma unroll
                        for (int e = 0; e < 2; ++e) s[e] = mfma_bf16(wh, v[e].m, s[e]);
#pragma unroll
                        for (int e = 0; e < 2; ++e) part[e][o] = mfma_bf16(wh, v[e].h, part[e][o]);
#pragma unroll
                        for (int e = 0; e < 2; ++e) part[e][o] += s[e];
                    }
                }
                const int yo = a - 3;
                if (yo >= r0) {
                    // lane (i, q): part[e][o][2] = filter column dx = q at column 2i + e, which belongs to
                    // output column 2i + e + 1 - q
                    float2 held;
#pragma unroll
                    for (int o = 0; o < 2; ++o) {
                        const float z0 = part[0][o][2], z1 = part[1][o][2];
                        const float l1 = from_left(z1), r0v = from_right(z0);
                        const float d0 = sum_lane_column(q == 0 ? l1 : q == 1 ? z0 : q == 2 ? z1 : bias4[o]);
                        const float d1 = sum_lane_column(q == 0 ? z0 : q == 1 ? z1 : q == 2 ? r0v : bias4[o]);
                        held.x = o == 0 || q != 0 ? d0 : held.x;
                        held.y = o == 0 || q != 0 ? d1 : held.y;
                    }
                    // the parts of the columns before (side 0) and after the wavefront's, in the lanes that hold them
                    int ln = lane;
                    asm volatile("" : "+v"(ln));
                    s_held[64 * wave + ln] = held;
                    if (ln == 32 || ln == 15) {
                        const int side = ln == 32 ? 0 : 1;
                        const float z[2] = { side ? part[1][0][2] : part[0][0][2], side ? part[1][1][2] : part[0][1][2] };
                        s_side[yo & 1][wave][2 * side] = z[0];
                        s_side[yo & 1][wave][2 * side + 1] = z[1];
                        if (side ? wave == kWaves - 1 && strip + 1 < strips : wave == 0 && strip > 0) {
                            float* to = edge + (((int64_t)(strip - 1 + side) * 2 + side) * G + yo) * 2;
                            to[0] = z[0];
                            to[1] = z[1];
                        }
                    }
                }
            }
        }
        if (active && a <= r1 + 1) rc.stages<0, kTail>(c2, c0, c1);
        lds_copies_arrived();  // the row has arrived
        __syncthreads();
    };
    Acc c0, c1, c2;
    for (int pos = 0; pos < 4; ++pos)
        for (int nb = 0; nb < 2; ++nb) c0[pos][nb] = c1[pos][nb] = c2[pos][nb] = v4f{ 0.f, 0.f, 0.f, 0.f };
    for (int a = r0 - 2; a <= r1 + 2; a += 3) {
        step(a, c0, c1, c2);
        if (a + 1 <= r1 + 2) step(a + 1, c2, c0, c1);
        if (a + 2 <= r1 + 2) step(a + 2, c1, c2, c0);
    }
    if (active) finish(r1 - 1);
}

// The columns on the two sides of a strip boundary miss one filter column each: the part that the
// neighbouring strip's block computed.  edge[b][side][y][o]: boundary b, side 0 for the column before it.
static __global__ void k_strip_edges(int32_t G, const float* __restrict__ edge, float* __restrict__ disp)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= (int64_t)((G + SW - 1) / SW - 1) * 4 * G) return;
    const int o = (int)(k & 1);
    const int64_t row = k >> 1;  // (b * 2 + side) * G + y
    const int y = (int)(row % G), side = (int)(row / G) & 1;
    const int x = (int)(row / (2 * (int64_t)G) + 1) * SW - 1 + side;
    if (x < G) disp[(int64_t)o * G * G + (int64_t)y * G + x] += edge[k];
}

inline size_t workspace_bytes(int32_t G)
{
    return kOffEdge + edge_bytes(G) + sizeof(float) * (size_t)C * (size_t)G * (size_t)G;
}

inline void forward(int32_t G, const float* vel, const cnnsns_cnn& w, float* disp, void* ws, int cus,
                    hipStream_t stream)
{
    char* base = static_cast<char*>(ws);
    float* edge = reinterpret_cast<float*>(base + kOffEdge);
    float* act2 = reinterpret_cast<float*>(base + kOffEdge + edge_bytes(G));
    const RowPlan plan = row_plan(G, cus);
    const unsigned grid = (unsigned)(plan.blocks() + 7) / 8 * 8;
    k_rows_prep<<<(kRowsPrepItems + 255) / 256, 256, 0, stream>>>(w.w[0], w.w[1], w.w[2], w.w[3], base);
    k_rows12_f32<<<grid, kThreads, 0, stream>>>(G, plan, vel, base, w.b[0], w.b[1], act2);
    k_rows34_f32<<<grid, kThreads, 0, stream>>>(G, plan, act2, base, w.b[2], w.b[3], edge, disp);
    if (plan.strips > 1)
        k_strip_edges<<<(unsigned)(((int64_t)(plan.strips - 1) * 4 * G + 255) / 256), 256, 0, stream>>>(G, edge, disp);
}

}  // namespace rows
}  // namespace cnnsns
