// The paper's classifier CNN (Sec. 2.3, eq. 7-8): the prediction step of
// Alg. 2 as a per-particle multiclass classification, in 2D on the overlay.
//
// Input preparation (Sec. 2.3).  Elements are represented by their centroids
// (vertices summed in ascending node id, then divided by 3); the ASG filter
// assigns each element to the overlay cell holding its centroid, and average
// pooling gives every cell the mean of its elements' centroids (summed in
// ascending element id), or the cell centre when it has none.  This grid is
// built once per mesh.  For a point x_p the filtered region is the 9 x 9 block
// of cells centred on the cell of x_p, extended at the grid boundary by the
// nearest cell (the padding layer); its input is G (pooled centroid - x_p) per
// cell, and x_p's own offset in its cell, x_p G - (cell + 1/2).  Both are
// formed in FP64 and rounded to FP32.
//
// Network (FP32 weights in PyTorch layouts): module 1, conv 3x3 2 -> 16, ReLU,
// conv 3x3 16 -> 16, ReLU, 2 x 2 average pooling (4 x 4, flattened
// [channel][row][col]); module 2, FC 2 -> 256, ReLU, FC 256 -> 256, ReLU; then
// FC 512 -> 512, ReLU, and FC 512 -> 81: the logits.  The class is the argmax
// of the logits (the softmax of eq. 7 is monotone, so it has the same
// argmax), the lowest class on ties; class (dy + 4) 9 + (dx + 4) is the window
// cell at offset (dx, dy) and K_p is that cell's overlay lookup element.
//
// On the GPU: one wavefront per particle for module 1 (window gather, both
// convolutions on the matrix cores, pooling) and module 2's first layer; the three wide FC layers as
// batched matrix products over a chunk of particles, FP32 values as three BF16 ones (split.h); then the argmax and
// start.
#pragma clang fp contract(off)

#include <hipcub/hipcub.hpp>

#include "common.h"
#include "lds_copy.h"
#include "split.h"

namespace cnnsns {
namespace {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kW = 9, kR = 4, kNA = kW * kW;  // window side, radius, classes
constexpr int kC = 16;                         // conv channels
constexpr int kPW = kW + 2;                    // the window with a one-cell zero border (conv1's padding)
constexpr int kNF = kC * 4 * 4;                // module 1 features (256)
constexpr int kH1 = 256, kH2 = 512, kNZ = kNF + kH1;
constexpr int kBlock = 256;
constexpr int64_t kChunk = 65536;  // particles per pass of the fully connected layers

__device__ __forceinline__ int32_t cell_of(double x, int32_t G)
{
    const double f = floor(x * (double)G);
    if (!(f >= 0.0)) return 0;  // negative or NaN
    if (f > (double)(G - 1)) return G - 1;
    return (int32_t)f;
}

__device__ __forceinline__ int32_t clamp_cell(int32_t c, int32_t G)
{
    return c < 0 ? 0 : (c >= G ? G - 1 : c);
}

// centroid of element t with its vertices summed in ascending node id
__device__ __forceinline__ void centroid_by_id(const ElemRec* __restrict__ rec, const int32_t* __restrict__ tri,
                                               int64_t t, double& x, double& y)
{
    const ElemRec r = rec[t];
    int32_t id[3] = { tri[3 * t], tri[3 * t + 1], tri[3 * t + 2] };
    double px[3] = { r.ax, r.bx, r.cx }, py[3] = { r.ay, r.by, r.cy };
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2 - i; ++j)
            if (id[j] > id[j + 1]) {
                const int32_t s = id[j];
                id[j] = id[j + 1];
                id[j + 1] = s;
                const double sx = px[j], sy = py[j];
                px[j] = px[j + 1];
                py[j] = py[j + 1];
                px[j + 1] = sx;
                py[j + 1] = sy;
            }
    x = ((px[0] + px[1]) + px[2]) / 3.0;
    y = ((py[0] + py[1]) + py[2]) / 3.0;
}

// pass 1 of the pooled grid: each element's cell (the sort key) and the cell counts
__global__ void k_pool_cells(int64_t n_tri, const ElemRec* __restrict__ rec, const int32_t* __restrict__ tri,
                             int32_t G, uint32_t* __restrict__ key, int32_t* __restrict__ val,
                             uint32_t* __restrict__ count)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n_tri) return;
    double x, y;
    centroid_by_id(rec, tri, t, x, y);
    const uint32_t c = (uint32_t)cell_of(y, G) * (uint32_t)G + (uint32_t)cell_of(x, G);
    key[t] = c;
    val[t] = (int32_t)t;
    atomicAdd(&count[c], 1u);
}

// pass 2: per cell, the mean of its elements' centroids in ascending element id (the stable sort keeps the
// ids of a cell ascending), or the cell centre
__global__ void k_pool_mean(int32_t G, const ElemRec* __restrict__ rec, const int32_t* __restrict__ tri,
                            const int32_t* __restrict__ sorted, const uint32_t* __restrict__ first,
                            const uint32_t* __restrict__ count, double2* __restrict__ pool)
{
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= (int64_t)G * G) return;
    const uint32_t k0 = first[c], k = count[c];
    double2 p;
    if (k == 0) {
        p.x = ((double)(c % G) + 0.5) / (double)G;
        p.y = ((double)(c / G) + 0.5) / (double)G;
    } else {
        double sx = 0.0, sy = 0.0;
        for (uint32_t q = 0; q < k; ++q) {
            double x, y;
            centroid_by_id(rec, tri, sorted[k0 + q], x, y);
            sx += x;
            sy += y;
        }
        p.x = sx / (double)k;
        p.y = sy / (double)k;
    }
    pool[c] = p;
}

// Module 1 and module 2's first layer, one wavefront per particle (persistent blocks).  conv1 (K = 18) runs on
// the FP32 matrix instruction, all 81 cells; its output is split into three BF16 parts in LDS (split.h) and conv2
// runs on those, K = 32 being two taps of 16 channels, for the 64 cells that the 2 x 2 pooling reads (the ninth
// row and column are dropped): four blocks of 16, one for each place in a 2 x 2 pool, so that a lane holds all
// four cells of its pool and averages them in registers.  Twelve wavefronts, three per SIMD, share conv2's
// operands in LDS (kept in registers they spilled).
//
// What bounds it: matrix instructions (30 of 32 cycles and 120 of 16 a particle) and vector instructions, which add
// up on a SIMD (cnn_rows.h).  With conv2 on the FP32 instruction over 96 cells, each of its accumulators written back
// for the pooling, 65,536 particles took 364 us; now 150.  At three wavefronts per SIMD two registers still spill.
constexpr int kMThreads = 768;
constexpr int kMW = kW + 1;              // conv2's input: the window with a border of one, less the last row and column
constexpr int kMPart = kMW * kMW * 2;    // bf16x8 of one part: two chunks of eight channels a cell

// A cell's place, rows and columns from the border: even columns first, then the odd ones.  A lane of conv2 reads
// every second cell, and a 16-lane group of a 16-byte read (lanes 0-7 with 56-63, ...) then covers 128 bytes
// of two rows, at the two chunks of a cell: sixteen distinct places of the 64 banks.
__host__ __device__ constexpr int m_place(int row, int c)
{
    return row * kMW + (c >> 1) + (c & 1) * (kMW / 2);
}

__global__ __launch_bounds__(kMThreads) __attribute__((amdgpu_waves_per_eu(3, 3))) void k_cls_module1(
    int64_t n, const double2* __restrict__ xp, int32_t G, const double2* __restrict__ pool,
    const float* __restrict__ w1, const float* __restrict__ b1, const float* __restrict__ w2,
    const float* __restrict__ b2, const float* __restrict__ wx1, const float* __restrict__ bx1,
    float* __restrict__ z, int ldz, float* __restrict__ m1, int ldm)
{
    constexpr int kWaves = kMThreads / 64;
    __shared__ bf16x8 s_a1[kWaves][3 * kMPart];
    __shared__ bf16x8 s_w2[5 * 3 * 64];
    __shared__ float s_in[kWaves][2][kPW * kPW];
    __shared__ v4f s_x1[kH1 * 3 / 4];  // module 2's first layer: w0, w1, bias, kH1 of each

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int i = lane & 15, q = lane >> 4;
    for (int j = tid; j < kH1; j += kMThreads) {
        float* x1 = reinterpret_cast<float*>(s_x1);
        x1[j] = wx1[2 * j];
        x1[kH1 + j] = wx1[2 * j + 1];
        x1[2 * kH1 + j] = bx1[j];
    }
    float* in = &s_in[wave][0][0];
    bf16x8* a1 = &s_a1[wave][0];
    for (int k = lane; k < 2 * kPW * kPW; k += 64) in[k] = 0.f;
    const bf16x8 none = __builtin_bit_cast(bf16x8, u32x4{ 0, 0, 0, 0 });
    for (int k = lane; k < 3 * kMPart; k += 64) a1[k] = none;
    // conv2's A operands: row = output channel l%16; lane group g of K step st takes tap 2 st + g/2 (zero past the
    // ninth), channels 8 (g%2) + j
    for (int k = tid; k < 5 * 3 * 64; k += kMThreads) {
        const int l = k & 63, part = (k >> 6) % 3, t = 2 * (k / 192) + (l >> 5), c = 8 * ((l >> 4) & 1);
        bf16x8 v;
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = split_part(t < 9 ? w2[((l & 15) * kC + c + j) * 9 + t] : 0.f, part);
        s_w2[k] = v;
    }
    __syncthreads();  // the weights, and the zero borders, which no point's writes touch
    // a wavefront takes points p, p + the grid's wavefront count, ...: its window and conv1 output are its
    // own LDS regions, so only the wavefront's own accesses need ordering
    auto wave_sync = [] {
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    // conv1: A operands (row = output channel i, k = 4 st + q = 9 ci + tap, zero for k >= 18) and the offsets of
    // their inputs; the lane's cell of each 16-cell block (the last block repeats cell 80): where its window starts
    // and where its result goes
    float w1k[5];
    int off1[5], base[6], to[6];
#pragma unroll
    for (int st = 0; st < 5; ++st) {
        const int k = min(4 * st + q, 17), t = k % 9;
        w1k[st] = 4 * st + q < 18 ? w1[i * 18 + k] : 0.f;
        off1[st] = (k / 9) * kPW * kPW + (t / 3) * kPW + t % 3;
    }
#pragma unroll
    for (int mb = 0; mb < 6; ++mb) {
        const int px = min(mb * 16 + i, kNA - 1), r = px / kW, c = px % kW;
        base[mb] = r * kPW + c;
        to[mb] = m_place(r + 1, c + 1);
    }
    // where the lane's pool i reads the tap of conv2's K step st, 2 st + q / 2, for the left and right cells of
    // its upper row (the tenth tap has zero weights and reads the ninth's cell)
    int at[5][2];
#pragma unroll
    for (int st = 0; st < 5; ++st)
#pragma unroll
        for (int dx = 0; dx < 2; ++dx) {
            const int t = min(2 * st + (q >> 1), 8);
            at[st][dx] = m_place(2 * (i >> 2) + t / 3, 2 * (i & 3) + dx + t % 3) * 2 + (q & 1);
        }
    v4f bias1, bias2;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        bias1[r] = b1[4 * q + r];
        bias2[r] = b2[4 * q + r];
    }

    // the window's pooled values of the wavefront's next particle are gathered into registers while
    // the current one computes (lane o holds window cells o and o + 64)
    const int64_t stride = (int64_t)gridDim.x * kWaves;
    double2 pn = double2{ 0.0, 0.0 };
    double2 qn[2] = { double2{ 0.0, 0.0 }, double2{ 0.0, 0.0 } };
    auto gather = [&](int64_t k) {
        pn = xp[k];
        const int32_t gx = cell_of(pn.x, G), gy = cell_of(pn.y, G);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int o = lane + 64 * u;
            if (o < kNA) {
                const int dy = o / kW - kR, dx = o % kW - kR;
                qn[u] = pool[(int64_t)clamp_cell(gy + dy, G) * G + clamp_cell(gx + dx, G)];
            }
        }
    };
    int64_t p0 = (int64_t)blockIdx.x * kWaves + wave;
    if (p0 < n) gather(p0);
    for (; p0 < n; p0 += stride) {
        const double2 p = pn;
        const int32_t cx = cell_of(p.x, G), cy = cell_of(p.y, G);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int o = lane + 64 * u;
            if (o < kNA) {
                const int at1 = (o / kW + 1) * kPW + (o % kW + 1);
                in[at1] = (float)((qn[u].x - p.x) * (double)G);
                in[kPW * kPW + at1] = (float)((qn[u].y - p.y) * (double)G);
            }
        }
        const float xo0 = (float)(p.x * (double)G - ((double)cx + 0.5));
        const float xo1 = (float)(p.y * (double)G - ((double)cy + 0.5));
        wave_sync();
        if (p0 + stride < n) gather(p0 + stride);
        {
            v4f acc[6];
#pragma unroll
            for (int mb = 0; mb < 6; ++mb) acc[mb] = bias1;
#pragma unroll
            for (int st = 0; st < 5; ++st)
#pragma unroll
                for (int mb = 0; mb < 6; ++mb)
                    acc[mb] = __builtin_amdgcn_mfma_f32_16x16x4f32(w1k[st], in[base[mb] + off1[st]], acc[mb], 0, 0, 0);
            // lane: channels 4q + r of its cell
#pragma unroll
            for (int mb = 0; mb < 6; ++mb) {
                u32x2 h, m, l;
                uint32_t ph, pm, pl;
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    split_pair(fmaxf(acc[mb][2 * j], 0.f), fmaxf(acc[mb][2 * j + 1], 0.f), ph, pm, pl);
                    h[j] = ph;
                    m[j] = pm;
                    l[j] = pl;
                }
                u32x2* dst = reinterpret_cast<u32x2*>(a1) + to[mb] * 4 + q;
                dst[0] = h;
                dst[2 * kMPart] = m;
                dst[4 * kMPart] = l;
            }
        }
        wave_sync();
        v4f hi[4], lo[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            hi[m] = bias2;
            lo[m] = v4f{ 0.f, 0.f, 0.f, 0.f };
        }
#pragma unroll
        for (int st = 0; st < 5; ++st) {
            bf16x8 x[4][3];
#pragma unroll
            for (int m = 0; m < 4; ++m)  // m = 2 dy + dx
#pragma unroll
                for (int part = 0; part < 3; ++part)
                    x[m][part] = a1[at[st][m & 1] + (m >> 1) * kMW * 2 + part * kMPart];
            bf16x8 w[3];
#pragma unroll
            for (int part = 0; part < 3; ++part) w[part] = s_w2[(st * 3 + part) * 64 + lane];
            constexpr int wp[6] = { 0, 0, 1, 1, 0, 2 }, xq[6] = { 0, 1, 0, 1, 2, 0 };
#pragma unroll
            for (int k = 0; k < 6; ++k)
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    v4f& acc = k == 0 ? hi[m] : lo[m];
                    acc = mfma_bf16(w[wp[k]], x[m][xq[k]], acc);
                }
        }
        // 2 x 2 average pooling, [channel][row][col] order
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float y[4];
#pragma unroll
            for (int m = 0; m < 4; ++m) y[m] = fmaxf(hi[m][r] + lo[m][r], 0.f);
            z[p0 * ldz + (4 * q + r) * 16 + i] = (((y[0] + y[1]) + y[2]) + y[3]) * 0.25f;
        }
        // module 2, first layer: FC 2 -> 256 on x_p's offset, outputs 4 lane ..
        {
            const v4f wa = s_x1[lane], wb = s_x1[kH1 / 4 + lane], bx = s_x1[kH1 / 2 + lane];
            v4f v;
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = fmaxf(bx[r] + wa[r] * xo0 + wb[r] * xo1, 0.f);
            *reinterpret_cast<v4f*>(m1 + p0 * ldm + 4 * lane) = v;
        }
        wave_sync();  // the next point's window and conv1 output replace these
    }
}

// The wide fully connected layers, C[m][n] = act(bias[n] + sum_k A[m][k] W[n][k]) for m < M, on the BF16 matrix
// instruction with both operands as three BF16 values (split.h).  A block takes BM particles x BN outputs; a
// wavefront MB x NB blocks of 16 x 16 (rows = outputs, columns = particles, so a lane ends with four consecutive
// outputs of a particle), the products of the high parts and the small ones in accumulators of their
// own.  K goes in slices of 32, KS of them a step, double-buffered in LDS: the weights' operands are copied straight
// into LDS as prepared (k_cls_prep), the activations are loaded into registers, split and written after the step's
// products.  Small tiles, whose steps are latency and not products, take two slices a step.
//
// What bounds it: matrix instructions, 96 per wavefront and slice (16.5 cycles each) at 128 x 256, 1.5 us of the
// 2.8 a slice takes; the rest is the splitting, the LDS reads and the barrier, which one block per compute unit
// does not hide.  65,536 particles, 512 -> 512: 0.18 ms, 0.36 on the FP32 instruction in 128 x 128 tiles.  One kernel
// for all three layers with the activations passed on already split took 0.30 ms against 0.31 for the three, and
// 69 us against 46 at 300 particles, where a block's serial chain of slices is all that counts.
constexpr int kDenseThreads = 512;

// Operand-ordered split weights of a layer with N (padded to 16) outputs and K inputs:
// ws[((ks * (N / 16) + n16) * 3 + part) * 64 + l][j] = that part of W[16 n16 + l%16][32 ks + 8 (l/16) + j].
__device__ __forceinline__ void dense_prep(int k, int N, int K, int n_real, const float* __restrict__ w,
                                           bf16x8* __restrict__ ws)
{
    const int l = k & 63, part = (k >> 6) % 3, blk = k / 192, n16 = blk % (N / 16), ks = blk / (N / 16);
    const int n = 16 * n16 + (l & 15), k0 = 32 * ks + 8 * (l >> 4);
    bf16x8 v;
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = split_part(n < n_real ? w[(int64_t)n * K + k0 + j] : 0.f, part);
    ws[k] = v;
}
constexpr int kNL = 96;                                  // the 81 logits padded to six blocks
constexpr int kD1 = kH1 / 16 * (kH1 / 32) * 192;         // bf16x8 of the three layers
constexpr int kD2 = kH2 / 16 * (kNZ / 32) * 192;
constexpr int kD3 = kNL / 16 * (kH2 / 32) * 192;

__global__ void k_cls_prep(const float* __restrict__ w3, const float* __restrict__ w4, const float* __restrict__ w5,
                           bf16x8* __restrict__ ws)
{
    int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < kD1) return dense_prep(k, kH1, kH1, kH1, w3, ws);
    if ((k -= kD1) < kD2) return dense_prep(k, kH2, kNZ, kH2, w4, ws + kD1);
    if ((k -= kD2) < kD3) dense_prep(k, kNL, kH2, kNA, w5, ws + kD1 + kD2);
}

// One part of BM rows of 32 inputs in LDS: four 16-byte chunks of eight a row, chunk c of row r at place
// c ^ 2 (r / 4 mod 2).  The LDS serves a 16-byte read in groups of 16 lanes over 64 four-byte banks, a group
// joining lanes 0-7 with 56-63 (8-15 with 48-55, ...): here eight consecutive rows at chunk c and the next eight
// at chunk 3 - c.  Eight rows take each place of a 256-byte line of four rows twice, r / 4 odd and even, which
// the exchange puts on chunks c and c ^ 2, and 3 - c has the other parity: sixteen distinct banks.
__device__ __forceinline__ int dense_slot(int r, int c)
{
    return r * 4 + (c ^ ((r >> 1) & 2));
}

// N outputs, of which n_real exist (rows of C hold ldc; with VEC all exist and a lane's four are stored at once)
template <int MB, int NB, int WM, int WN, int KS, bool RELU, bool VEC>
__global__ __launch_bounds__(kDenseThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_dense_split(
    int M, int N, int n_real, int K, const float* __restrict__ A, int lda, const bf16x8* __restrict__ ws,
    const float* __restrict__ bias, float* __restrict__ Cm, int ldc)
{
    static_assert(WM * WN * 64 == kDenseThreads, "eight wavefronts");
    constexpr int BM = 16 * MB * WM, BN = 16 * NB * WN, NF = BN / 16 * 3;  // weight operands of a slice
    constexpr int PER = BM * 8 / kDenseThreads;
    static_assert(BM * 8 % kDenseThreads == 0, "whole rounds of activation loads");
    __shared__ bf16x8 s_w[2][KS][NF * 64];
    __shared__ bf16x8 s_x[2][KS][3 * BM * 4];
    const int m0 = blockIdx.x * BM, n0 = blockIdx.y * BN;
    const int tid = threadIdx.x, lane = tid & 63, i = lane & 15, q = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave / WN, wn = wave % WN;

    // weights of step ks (KS slices) straight into LDS, one operand (64 lanes x 16 bytes) a wavefront instruction
    auto load_w = [&](int ks) {
        const bf16x8* src = ws + ((int64_t)ks * KS * (N / 16) + n0 / 16) * 192 + lane;
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int k = 0; k < (NF + 7) / 8; ++k) {  // no loop: a taken branch costs some 40 cycles
                const int f = wave + 8 * k;
                if (8 * (k + 1) <= NF || f < NF) lds_copy16(src + s * (N / 16) * 192 + f * 64, s_w[ks & 1][s] + f * 64);
            }
    };
    v4f pa[KS][PER];
    auto fetch = [&](int ks) {
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int h = 0; h < PER; ++h) {
                const int e = tid + h * kDenseThreads, r = min(m0 + (e >> 3), M - 1);  // rows past M: not stored
                pa[s][h] = *reinterpret_cast<const v4f*>(A + (int64_t)r * lda + 32 * (ks * KS + s) + 4 * (e & 7));
            }
    };
    auto stash = [&](int ks) {
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int h = 0; h < PER; ++h) {
                const int e = tid + h * kDenseThreads;
                u32x2 p[3];
                uint32_t a, b, c;
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    split_pair(pa[s][h][2 * j], pa[s][h][2 * j + 1], a, b, c);
                    p[0][j] = a;
                    p[1][j] = b;
                    p[2][j] = c;
                }
                u32x2* to = reinterpret_cast<u32x2*>(s_x[ks & 1][s] + dense_slot(e >> 3, (e & 7) >> 1)) + (e & 1);
#pragma unroll
                for (int part = 0; part < 3; ++part) to[part * BM * 8] = p[part];
            }
    };
    v4f hi[MB][NB], lo[MB][NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        v4f b;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int n = n0 + 16 * (wn * NB + nb) + 4 * q + r;
            b[r] = VEC || n < n_real ? bias[n] : 0.f;
        }
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            hi[mb][nb] = b;
            lo[mb][nb] = v4f{ 0.f, 0.f, 0.f, 0.f };
        }
    }
    load_w(0);
    fetch(0);
    stash(0);
    lds_copies_arrived();  // the weights have arrived
    __syncthreads();
    const int steps = K / (32 * KS);
    auto products = [&](int ks) {
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const bf16x8* sw = s_w[ks & 1][s] + wn * NB * 192 + lane;
            const bf16x8* sx = s_x[ks & 1][s];
            bf16x8 w[NB][3], x[MB][3];
#pragma unroll
            for (int part = 0; part < 3; ++part) {
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) w[nb][part] = sw[(nb * 3 + part) * 64];
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) x[mb][part] = sx[part * BM * 4 + dense_slot(16 * (wm * MB + mb) + i, q)];
            }
            constexpr int wp[6] = { 0, 0, 1, 1, 0, 2 }, xp[6] = { 0, 1, 0, 1, 2, 0 };
#pragma unroll
            for (int k = 0; k < 6; ++k)
#pragma unroll
                for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) {
                        v4f& acc = k == 0 ? hi[mb][nb] : lo[mb][nb];
                        acc = mfma_bf16(w[nb][wp[k]], x[mb][xp[k]], acc);
                    }
        }
    };
    // The last step apart, so that no load is pending where the loop starts again: the compiler would wait for it
    // there, and with it for the copies just issued.
    for (int ks = 0; ks + 1 < steps; ++ks) {
        load_w(ks + 1);  // these land while the step's products issue
        fetch(ks + 1);
        __builtin_amdgcn_sched_barrier(0);
        products(ks);
        if (KS > 1) __builtin_amdgcn_sched_barrier(0);  // few products: none wait for the activations
        stash(ks + 1);
        lds_copies_arrived();
        __syncthreads();
    }
    products(steps - 1);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
        const int m = m0 + 16 * (wm * MB + mb) + i;
        if (m >= M) continue;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const int n = n0 + 16 * (wn * NB + nb) + 4 * q;
            v4f v = hi[mb][nb] + lo[mb][nb];
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = RELU ? fmaxf(v[r], 0.f) : v[r];
            float* to = Cm + (int64_t)m * ldc + n;
            if (VEC) {
                *reinterpret_cast<v4f*>(to) = v;
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (n + r < n_real) to[r] = v[r];
            }
        }
    }
}

// The layer on M particles: 128 x 256 tiles while they fill the chip, 128 x 64 tiles for a last round that would
// leave most compute units idle.  A round of the large tiles takes 45 us (512 -> 512), one of the small ones, four
// times as many blocks, 14: the small ones are the faster up to three rounds.
template <bool RELU>
void dense(int M, int N, int K, const float* A, int lda, const bf16x8* ws, const float* bias, float* Cm, int ldc,
           unsigned cus, hipStream_t stream)
{
    const unsigned mt = (unsigned)((M + 127) / 128), nb = (unsigned)N / 256;
    unsigned large = mt - mt % std::max(cus / nb, 1u);  // row tiles in whole rounds
    if ((mt - large) * 4 * nb > 3 * cus) large = mt;
    const int rows = (int)std::min<unsigned>(large * 128, (unsigned)M);
    if (large)
        k_dense_split<4, 4, 2, 4, 1, RELU, true><<<dim3(large, nb), kDenseThreads, 0, stream>>>(rows, N, N, K, A, lda, ws, bias, Cm, ldc);
    if (large < mt)
        k_dense_split<2, 2, 4, 2, 2, RELU, true><<<dim3(mt - large, N / 64), kDenseThreads, 0, stream>>>(
            M - rows, N, N, K, A + (int64_t)rows * lda, lda, ws, bias, Cm + (int64_t)rows * ldc, ldc);
}

// The last layer, 512 -> 81, in the same way: 128-row blocks in whole rounds, and 64-row blocks, two slices a step, for a
// last round that these cover at once (300 particles: 12 us against 20 with 128 rows; 65,536: 62 against 57).
void dense_logits(int M, const float* A, const bf16x8* ws, const float* bias, float* L, unsigned cus, hipStream_t stream)
{
    const unsigned mt = (unsigned)((M + 127) / 128);
    unsigned large = mt - mt % cus;
    if ((mt - large) * 2 > cus) large = mt;
    const int rows = (int)std::min<unsigned>(large * 128, (unsigned)M), rest = M - rows;
    if (large)
        k_dense_split<2, 3, 4, 2, 1, false, false><<<large, kDenseThreads, 0, stream>>>(rows, kNL, kNA, kH2, A, kH2, ws, bias, L, kNA);
    if (rest)
        k_dense_split<1, 3, 4, 2, 2, false, false><<<(rest + 63) / 64, kDenseThreads, 0, stream>>>(
            rest, kNL, kNA, kH2, A + (int64_t)rows * kH2, kH2, ws, bias, L + (int64_t)rows * kNA, kNA);
}

// The argmax of each particle's logits (the lowest class on ties) and its start element: the lookup element
// of that window cell, else the fallback start, else element 0.
__global__ void k_cls_argmax(int64_t n, const double2* __restrict__ xp, int32_t G, const int32_t* __restrict__ lookup,
                             const float* __restrict__ logits, int ldl, const int32_t* __restrict__ fallback,
                             int32_t* __restrict__ start, int32_t* __restrict__ cls)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float* h = logits + i * ldl;
    int best = 0;
    float hb = h[0];
    for (int l = 1; l < kNA; ++l) {
        const float v = h[l];
        if (v > hb) {
            hb = v;
            best = l;
        }
    }
    const double2 p = xp[i];
    const int32_t cx = clamp_cell(cell_of(p.x, G) + best % kW - kR, G);
    const int32_t cy = clamp_cell(cell_of(p.y, G) + best / kW - kR, G);
    int32_t k = lookup[(int64_t)cy * G + cx];
    if (k < 0) k = fallback ? fallback[i] : 0;
    start[i] = k;
    if (cls) cls[i] = best;
}

inline unsigned blocks_for(int64_t n, int per)
{
    return (unsigned)((n + per - 1) / per);
}

// The pooled grid of a mesh, built on its first classification.
void build_pool(cnnsns_mesh_s& m, hipStream_t stream)
{
    const int64_t nt = m.n_tri, GG = (int64_t)m.G * m.G;
    if (GG > (int64_t)UINT32_MAX || nt > (int64_t)UINT32_MAX) fail(CNNSNS_EINVAL, "classify: overlay too large");
    void* tmp = nullptr;
    auto dmalloc = [&](size_t bytes) {
        void* p = nullptr;
        if (hipMalloc(&p, bytes ? bytes : 1) != hipSuccess) {
            (void)hipGetLastError();
            fail(CNNSNS_ENOMEM, "classify: pooled grid allocation of " + std::to_string(bytes) + " bytes");
        }
        return p;
    };
    struct Bufs {
        void* p[7] = {};
        ~Bufs()
        {
            for (void* q : p)
                if (q) (void)hipFree(q);
        }
    } b;
    auto* key = static_cast<uint32_t*>(b.p[0] = dmalloc(sizeof(uint32_t) * nt));
    auto* key2 = static_cast<uint32_t*>(b.p[1] = dmalloc(sizeof(uint32_t) * nt));
    auto* val = static_cast<int32_t*>(b.p[2] = dmalloc(sizeof(int32_t) * nt));
    auto* val2 = static_cast<int32_t*>(b.p[3] = dmalloc(sizeof(int32_t) * nt));
    auto* count = static_cast<uint32_t*>(b.p[4] = dmalloc(sizeof(uint32_t) * GG));
    auto* first = static_cast<uint32_t*>(b.p[5] = dmalloc(sizeof(uint32_t) * GG));
    auto* pool = static_cast<double2*>(dmalloc(sizeof(double2) * GG));
    try {
        hip_check(hipMemsetAsync(count, 0, sizeof(uint32_t) * GG, stream), "classify: pool counts");
        k_pool_cells<<<blocks_for(nt, kBlock), kBlock, 0, stream>>>(nt, m.rec, m.tri, m.G, key, val, count);
        int end_bit = 1;
        while (end_bit < 32 && ((uint64_t)1 << end_bit) < (uint64_t)GG) ++end_bit;
        size_t sort_bytes = 0, scan_bytes = 0;
        hip_check(hipcub::DeviceRadixSort::SortPairs(nullptr, sort_bytes, key, key2, val, val2, (int)nt, 0, end_bit,
                                                     stream),
                  "classify: sort size");
        hip_check(hipcub::DeviceScan::ExclusiveSum(nullptr, scan_bytes, count, first, (int)GG, stream),
                  "classify: scan size");
        tmp = b.p[6] = dmalloc(std::max(sort_bytes, scan_bytes));
        hip_check(hipcub::DeviceRadixSort::SortPairs(tmp, sort_bytes, key, key2, val, val2, (int)nt, 0, end_bit, stream),
                  "classify: sort");
        hip_check(hipcub::DeviceScan::ExclusiveSum(tmp, scan_bytes, count, first, (int)GG, stream), "classify: scan");
        k_pool_mean<<<blocks_for(GG, kBlock), kBlock, 0, stream>>>(m.G, m.rec, m.tri, val2, first, count, pool);
        hip_check(hipGetLastError(), "classify: pool kernels");
        hip_check(hipStreamSynchronize(stream), "classify: pooled grid");
    } catch (...) {
        (void)hipFree(pool);
        throw;
    }
    m.cls_pool = pool;
    m.device_bytes += (int64_t)(sizeof(double2) * GG);
}

}  // namespace

size_t cls_workspace_bytes(int64_t n)
{
    const int64_t ch = n < kChunk ? n : kChunk;
    return sizeof(bf16x8) * (size_t)(kD1 + kD2 + kD3) + sizeof(float) * (size_t)ch * (size_t)(kNZ + kH2 + kNA);
}

void run_classify(cnnsns_mesh_s& m, int64_t n, const double* xp, const cnnsns_cls& w, const int32_t* fallback,
                  int32_t* start, int32_t* cls, float* logits, hipStream_t stream)
{
    if (n == 0) return;
    std::lock_guard<std::mutex> lock(m.cls_ws.mu);
    if (!m.cls_pool) build_pool(m, stream);
    workspace_acquire(m.cls_ws, cls_workspace_bytes(n), stream, "classify");
    const int64_t ch = n < kChunk ? n : kChunk;
    bf16x8* wd = static_cast<bf16x8*>(m.cls_ws.ptr);   // the wide layers' weights
    float* Z = reinterpret_cast<float*>(wd + kD1 + kD2 + kD3);  // [ch][512]: module 1 | module 2
    float* Hb = Z + ch * kNZ;                          // [ch][512]: module 2's first layer, then FC h2
    float* Lw = Hb + ch * kH2;                         // [ch][81] logits when the caller keeps none
    const auto* xp2 = reinterpret_cast<const double2*>(xp);
    const unsigned cus = cnn_persistent_grid();
    k_cls_prep<<<(kD1 + kD2 + kD3 + kBlock - 1) / kBlock, kBlock, 0, stream>>>(w.w[3], w.w[4], w.w[5], wd);
    for (int64_t c0 = 0; c0 < n; c0 += ch) {
        const int mc = (int)(n - c0 < ch ? n - c0 : ch);
        float* L = logits ? logits + c0 * kNA : Lw;
        // persistent: one block per compute unit
        const unsigned mblocks = std::min<unsigned>(blocks_for(mc, kMThreads / 64), cus);
        k_cls_module1<<<mblocks, kMThreads, 0, stream>>>(
            mc, xp2 + c0, m.G, static_cast<const double2*>(m.cls_pool), w.w[0], w.b[0], w.w[1], w.b[1], w.w[2], w.b[2],
            Z, kNZ, Hb, kH2);
        dense<true>(mc, kH1, kH1, Hb, kH2, wd, w.b[3], Z + kNF, kNZ, cus, stream);
        dense<true>(mc, kH2, kNZ, Z, kNZ, wd + kD1, w.b[4], Hb, kH2, cus, stream);
        dense_logits(mc, Hb, wd + kD1 + kD2, w.b[5], L, cus, stream);
        k_cls_argmax<<<blocks_for(mc, kBlock), kBlock, 0, stream>>>(mc, xp2 + c0, m.G, m.lookup, L, kNA,
                                                                    fallback ? fallback + c0 : nullptr, start + c0,
                                                                    cls ? cls + c0 : nullptr);
    }
    hip_check(hipGetLastError(), "classify launch");
    workspace_used(m.cls_ws, stream);
}

}  // namespace cnnsns
