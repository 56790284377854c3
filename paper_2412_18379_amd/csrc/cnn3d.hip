// The displacement CNN in 3D (Sec. 2.3 with 3 x 3 x 3 kernels on a G x G x G
// overlay): 3 -> 32 -> 32 -> 32 -> 3 channels, zero padding of one cell, bias,
// ReLU after layers 1-3, FP32.
//
// All layers run as z-sweeps: a block owns a column of 8 x 32 cells and consecutive planes and keeps the input planes
// that its current outputs read, with their one-cell border, in LDS.  Layers 2 and 3 (32 -> 32, 94 % of the work) are
// dense contractions over 27 taps x 32 input channels per output cell on the matrix cores, with the weights as row
// operand and 16 consecutive cells along x as column operand, so that a lane ends with consecutive channels of
// one cell.  FP32 pass: layers 2 and 3 on BF16 instructions with three BF16 values per FP32 value (k3c_zsplit_f32,
// split.h), layer 1 (k3c_zconv1) and layer 4 (k3c_zconv4_f32) on the FP32 instruction.  BF16 pass (BF16 operands
// after layer 1, FP32 accumulation): layers 2-4 in k3c_zsweep_bf16, layer 4 with its 3 outputs padded to 16, layer 1
// with split operands (k3c_zconv1_split).
//
// Activations between layers: FP32 [G^3][32], cell-major (z, y, x; x fastest),
// 32 channels per cell.  Input velocity and output displacement: FP32
// [3][G][G][G] (component, z, y, x).
#include <mutex>

#include "common.h"
#include "split.h"

namespace cnnsns {
namespace {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float v8f __attribute__((ext_vector_type(8)));
typedef __bf16 bf16;
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

constexpr int C = 32;             // hidden channels
constexpr int CIO = 3;            // velocity / displacement components
constexpr int TAPS = 27;
constexpr int NWB = TAPS * 2 * 64;      // BF16 weights of one 32 -> 32 layer (bf16x8 entries)
constexpr int kBlock = 256;       // weight preparation

// BF16 operand-ordered weights: wb[(tap * 2 + nb) * 64 + l] holds, as 8 BF16 (rounded to
// nearest even), W[16 nb + l%16][8 (l/16) + j][tap] for j = 0..7: the A operand of
// v_mfma_f32_16x16x32_bf16 (row = output channel, k = input channel 8 (l/16) + j).
__device__ __forceinline__ void wprep_bf16(int k, const float* __restrict__ w, bf16x8* __restrict__ wb)
{
    const int l = k & 63, nb = (k >> 6) & 1, tap = k >> 7;
    const int o = 16 * nb + (l & 15), c0 = 8 * (l >> 4);
    v8f v;
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = w[(o * C + c0 + j) * TAPS + tap];
    wb[k] = __builtin_convertvector(v, bf16x8);
}

// Layer 4 in the BF16 pass on the matrix cores: the 3 output channels padded to one 16-row A
// block, wb4[tap * 64 + l] = W4[l%16][8 (l/16) + j][tap] as BF16 (zero for rows >= 3), so a tap is
// one v_mfma_f32_16x16x32_bf16 per 16 cells; lanes 0..15 receive output channels 0..3 of their
// cell, the first three of which are written with the bias added.
__device__ __forceinline__ void wprep4_bf16(int k, const float* __restrict__ w, bf16x8* __restrict__ wb)
{
    const int l = k & 63, tap = k >> 6;
    const int o = l & 15, c0 = 8 * (l >> 4);
    v8f v;
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = o < CIO ? w[(o * C + c0 + j) * TAPS + tap] : 0.f;
    wb[k] = __builtin_convertvector(v, bf16x8);
}

// Layers 2-4 of the BF16 pass as z-sweeps through LDS.  A block owns a column of ZY x ZX cells and zp consecutive
// planes (z_planes below), two of them a step: it keeps the four input planes that its two output planes read, each as a
// (ZY + 2) x (ZX + 2) slab with the one-cell border (zero outside the grid), and the two that the next step adds, in a
// ring in LDS, so every input cell is read from memory once per block (plus the borders) instead of once per tap.  The
// planes after these are loaded into registers while a step's taps run and written at the start of the next, to places
// that nothing reads then: one barrier a step.
//
// A tap is one v_mfma_f32_16x16x32_bf16 per 16 cells and 16 output channels.  Of the eight wavefronts each takes one
// half of the 32 output channels, its weights in registers, and 4 rows x 16 columns of both planes (32 -> 3, outputs
// padded to 16: 2 rows x 16 columns), so that an operand read from LDS feeds up to six (four) instructions.
//
// What bounds it: matrix instructions, 216 per wavefront and step at 32 -> 32 (7,130 cycles per SIMD), and the LDS, 72
// reads of a wavefront in that time (4,600 cycles).  With one plane a step, both halves in every wavefront and half of
// the weights read from LDS per tap it was the LDS, 162 reads for as many instructions, and two barriers a plane.  The
// three layers in us, before and now: G = 33: 33 and 31, 64: 50 and 47, 101: 218 and 178, 128: 310 and 258.
constexpr int ZY = 8, ZX = 32;                    // cells per block: rows, columns
constexpr int ZSY = ZY + 2, ZSX = ZX + 2;         // slab with its border
constexpr int ZRING = 6;                          // planes in LDS
constexpr int ZSLABB = ZSY * ZSX * 64;            // bytes of a slab
constexpr int kZThreads = 512;
constexpr int ZCHUNKS = ZSY * ZSX * 4;            // 16-byte pieces of a slab
constexpr int ZCH_PER_THREAD = (ZCHUNKS + kZThreads - 1) / kZThreads;
static_assert(ZY == 8 && ZX == 32 && kZThreads == 512, "the wavefronts' shares of a plane");

// Byte offset of 16-byte chunk c of slab cell i.  The LDS serves a 16-byte read in groups of 16 lanes over 64 four-byte
// banks, a group joining lanes 0-7 with 56-63 (8-15 with 48-55, ...): here eight consecutive cells at one chunk and
// eight others at the mirrored chunk, which the exchange puts on distinct banks.
__device__ __forceinline__ int zcell(int i, int c)
{
    return i * 64 + ((c ^ ((i >> 1) & 3)) << 4);
}

template <int NB>
__global__ __launch_bounds__(kZThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k3c_zsweep_bf16(
    int32_t G, int zp, const bf16* __restrict__ in, const bf16x8* __restrict__ wb, const float* __restrict__ bias,
    bf16* __restrict__ out, float* __restrict__ disp)
{
    constexpr int ROWS = 2 * NB;  // of a wavefront
    __shared__ __attribute__((aligned(16))) char s_slab[ZRING * ZSLABB];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, grp = lane >> 4;
    const int nb = NB == 2 ? wave & 1 : 0, part = NB == 2 ? wave >> 1 : wave;  // output half and share of the cells
    const int row0 = (part >> 1) * ROWS, col0 = 16 * (part & 1);
    const int tiles_x = (G + ZX - 1) / ZX, tiles_y = (G + ZY - 1) / ZY;
    const int64_t b = blockIdx.x;
    const int tx0 = (int)(b % tiles_x) * ZX, ty0 = (int)((b / tiles_x) % tiles_y) * ZY;
    const int z0 = (int)(b / ((int64_t)tiles_x * tiles_y)) * zp;
    const int z1 = min(z0 + zp, G);
    const int64_t GG = (int64_t)G * G;

    // This thread's pieces of a slab: byte offset in a plane of `in` (from a clamped position), whether the cell lies in
    // the grid, and the place in LDS
    uint32_t from[ZCH_PER_THREAD], keep[ZCH_PER_THREAD];
    int place[ZCH_PER_THREAD];
#pragma unroll
    for (int k = 0; k < ZCH_PER_THREAD; ++k) {
        const int e = min(tid + k * kZThreads, ZCHUNKS - 1), cell = e >> 2;
        const int gy = ty0 + cell / ZSX - 1, gx = tx0 + cell % ZSX - 1;
        keep[k] = gy >= 0 && gy < G && gx >= 0 && gx < G ? ~0u : 0u;
        from[k] = ((uint32_t)min(max(gy, 0), G - 1) * (uint32_t)G + (uint32_t)min(max(gx, 0), G - 1)) * (2 * C) + 16 * (e & 3);
        place[k] = zcell(cell, e & 3);
    }
    // Two planes p, p + 1 into registers: unconditional loads, so that they stay in flight while a step's taps run; the
    // zero padding is applied when they are stashed.
    u32x4 pf[2][ZCH_PER_THREAD];
    auto fetch = [&](int p) {
#pragma unroll
        for (int d = 0; d < 2; ++d) {
            const char* plane = reinterpret_cast<const char*>(in + (int64_t)min(max(p + d, 0), G - 1) * GG * C);
#pragma unroll
            for (int k = 0; k < ZCH_PER_THREAD; ++k) pf[d][k] = *reinterpret_cast<const u32x4*>(plane + from[k]);
        }
    };
    auto stash = [&](int p, int slot) {  // slot of p: even
#pragma unroll
        for (int d = 0; d < 2; ++d) {
            const uint32_t in_z = p + d >= 0 && p + d < G ? ~0u : 0u;
#pragma unroll
            for (int k = 0; k < ZCH_PER_THREAD; ++k)
                if ((k + 1) * kZThreads <= ZCHUNKS || tid + k * kZThreads < ZCHUNKS)
                    *reinterpret_cast<u32x4*>(s_slab + (slot + d) * ZSLABB + place[k]) = pf[d][k] & (keep[k] & in_z);
        }
    };
    fetch(z0 - 1);
    stash(z0 - 1, 0);
    fetch(z0 + 1);
    stash(z0 + 1, 2);
    fetch(z0 + 3);

    bf16x8 w[TAPS];
#pragma unroll
    for (int t = 0; t < TAPS; ++t) w[t] = wb[(t * NB + nb) * 64 + lane];
    v4f start{ 0.f, 0.f, 0.f, 0.f };  // 32 -> 3: the bias is added to the result
    if (NB == 2) start = *reinterpret_cast<const v4f*>(bias + 16 * nb + 4 * grp);

    // operand addresses in a slab: row r (0: above the wavefront's first), column dx; the exchange repeats after four rows
    // (34 cells each)
    int at[4][3];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int dx = 0; dx < 3; ++dx) at[r][dx] = zcell((row0 + r) * ZSX + col0 + col + dx, grp);
    const int gx = tx0 + col0 + col;
    const unsigned to = NB == 2 ? gx * C + 16 * nb + 4 * grp : gx;  // the lane's place in a row of the result
    __syncthreads();
    int slot = 0;  // of plane z - 1
    for (int z = z0; z < z1; z += 2) {
        const int slot2 = slot == 4 ? 0 : slot + 2, slot4 = slot == 0 ? 4 : slot - 2;
        stash(z + 3, slot4);
        fetch(z + 5);  // lands while this step computes (past the block's last planes: unused)
        __builtin_amdgcn_sched_barrier(0);  // the loads stay ahead of the step's taps
        v4f acc[2][ROWS];  // output plane, row
        // input plane z - 1 + p, row r, column dx, in the order in which every output's taps are summed
        constexpr int NG = 4 * (ROWS + 2) * 3, PF = 4;
        bf16x8 x[PF + 1];
        auto read = [&](int g) {
            const int p = g / (3 * (ROWS + 2)), r = g / 3 % (ROWS + 2), dx = g % 3;
            x[g % (PF + 1)] = *reinterpret_cast<const bf16x8*>(s_slab + ((p < 2 ? slot : slot2) + (p & 1)) * ZSLABB + at[r & 3][dx] +
                                                               (r >> 2) * 4 * ZSX * 64);
        };
#pragma unroll
        for (int g = 0; g < PF; ++g) read(g);
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const int p = g / (3 * (ROWS + 2)), r = g / 3 % (ROWS + 2), dx = g % 3;
            if (g + PF < NG) read(g + PF);
            __builtin_amdgcn_sched_barrier(0);  // the reads stay ahead of the instructions
#pragma unroll
            for (int oz = 0; oz < 2; ++oz)
#pragma unroll
                for (int oy = 0; oy < ROWS; ++oy) {
                    const int dz = p - oz, dy = r - oy;
                    if (dz < 0 || dz > 2 || dy < 0 || dy > 2) continue;
                    const int t = (dz * 3 + dy) * 3 + dx;
                    acc[oz][oy] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[t], x[g % (PF + 1)], t == 0 ? start : acc[oz][oy], 0, 0, 0);
                }
        }
        // results: lane (col, grp) holds rows 4 grp + j (output channels 16 nb + 4 grp + j) of cell col
        auto emit = [&](int oz, int oy) {
            const int64_t row = (int64_t)(z + oz) * GG + (int64_t)(ty0 + row0 + oy) * G;
            const v4f a = acc[oz][oy];
            if (NB == 2) {
                const v4f v{ fmaxf(a.x, 0.f), fmaxf(a.y, 0.f), fmaxf(a.z, 0.f), fmaxf(a.w, 0.f) };
                *reinterpret_cast<bf16x4*>(out + row * C + to) = __builtin_convertvector(v, bf16x4);
            } else {
                disp[row + to] = a.x + bias[0];
                disp[GG * G + row + to] = a.y + bias[1];
                disp[2 * GG * G + row + to] = a.z + bias[2];
            }
        };
        if (gx < G && (NB == 2 || grp == 0)) {
            const int rows = min(ROWS, G - ty0 - row0);
            if (rows == ROWS && z + 1 < z1) {  // without a branch a row
#pragma unroll
                for (int k = 0; k < 2 * ROWS; ++k) emit(k / ROWS, k % ROWS);
            } else {
#pragma unroll
                for (int k = 0; k < 2 * ROWS; ++k)
                    if (k % ROWS < rows && z + k / ROWS < z1) emit(k / ROWS, k % ROWS);
            }
        }
        slot = slot2;
        __syncthreads();
    }
}

// Layer 1 of the FP32 pass (3 -> 32) as a z-sweep on the FP32 matrix instruction: the velocity's
// three planes in LDS as (u, v, w, 0) per cell, one v_mfma_f32_16x16x4f32 per tap and 16 output
// channels with K = the three components and a zero, the weights (one float per lane, tap and
// block of 16 output channels) held in registers.
constexpr int Z1CS = 4;  // floats per slab cell

constexpr int kZ1Threads = 1024;  // one 16-cell M-block per wavefront
__global__ __launch_bounds__(kZ1Threads) void k3c_zconv1(int32_t G, int zp, const float* __restrict__ vel,
                                                        const float* __restrict__ w, const float* __restrict__ bias,
                                                        float* __restrict__ out)
{
    constexpr int NCELL = ZSY * ZSX;
    static_assert(NCELL <= kZ1Threads && ZY * ZX == (kZ1Threads / 64) * 16, "one slab cell per thread");
    __shared__ __attribute__((aligned(16))) float s_v[3 * NCELL * Z1CS];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int col = lane & 15, grp = lane >> 4;
    // A operands: lane (col, grp) holds W[16 nb + col][grp][tap] (zero for grp = 3)
    float wa[TAPS][2];
#pragma unroll
    for (int t = 0; t < TAPS; ++t)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) wa[t][nb] = grp < CIO ? w[((16 * nb + col) * CIO + grp) * TAPS + t] : 0.f;
    const int tiles_x = (G + ZX - 1) / ZX, tiles_y = (G + ZY - 1) / ZY;
    const int64_t b = blockIdx.x;
    const int tx0 = (int)(b % tiles_x) * ZX, ty0 = (int)((b / tiles_x) % tiles_y) * ZY;
    const int z0 = (int)(b / ((int64_t)tiles_x * tiles_y)) * zp;
    const int z1 = min(z0 + zp, G);
    const int64_t GG = (int64_t)G * G, n = GG * G;
    const int r = wave >> 1, h = wave & 1;

    v4f pf;
    auto fetch = [&](int p) {  // thread tid < NCELL: its slab cell of plane p (zero outside the grid)
        pf = v4f{ 0.f, 0.f, 0.f, 0.f };
        if (tid < NCELL) {
            const int gy = ty0 + tid / ZSX - 1, gx = tx0 + tid % ZSX - 1;
            if (p >= 0 && p < G && gy >= 0 && gy < G && gx >= 0 && gx < G) {
                const int64_t c = (int64_t)p * GG + (int64_t)gy * G + gx;
                pf = v4f{ vel[c], vel[n + c], vel[2 * n + c], 0.f };
            }
        }
    };
    auto stash = [&](int p) {
        if (tid < NCELL) *reinterpret_cast<v4f*>(s_v + (((p + 3) % 3) * NCELL + tid) * Z1CS) = pf;
    };
    fetch(z0 - 1);
    stash(z0 - 1);
    fetch(z0);
    stash(z0);
    fetch(z0 + 1);
    stash(z0 + 1);
    __syncthreads();
    const v4f bl0 = *reinterpret_cast<const v4f*>(bias + 4 * grp);
    const v4f bl1 = *reinterpret_cast<const v4f*>(bias + 16 + 4 * grp);
    const int cell0 = r * ZSX + 16 * h + col;  // the lane's output cell in the slab, and its channel
    for (int z = z0; z < z1; ++z) {
        if (z + 2 < z1 + 1) fetch(z + 2);
        v4f acc0 = bl0, acc1 = bl1;
#pragma unroll
        for (int dz = 0; dz < 3; ++dz) {
            const float* sl = s_v + ((z + dz - 1 + 3) % 3) * NCELL * Z1CS + cell0 * Z1CS + grp;
#pragma unroll
            for (int t9 = 0; t9 < 9; ++t9) {
                const float a = sl[((t9 / 3) * ZSX + t9 % 3) * Z1CS];
                acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(wa[dz * 9 + t9][0], a, acc0, 0, 0, 0);
                acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(wa[dz * 9 + t9][1], a, acc1, 0, 0, 0);
            }
        }
        const int gy = ty0 + r, gx = tx0 + 16 * h + col;
        if (gy < G && gx < G) {
            float* dst = out + ((int64_t)z * GG + (int64_t)gy * G + gx) * C + 4 * grp;
            const v4f v0{ fmaxf(acc0.x, 0.f), fmaxf(acc0.y, 0.f), fmaxf(acc0.z, 0.f), fmaxf(acc0.w, 0.f) };
            const v4f v1{ fmaxf(acc1.x, 0.f), fmaxf(acc1.y, 0.f), fmaxf(acc1.z, 0.f), fmaxf(acc1.w, 0.f) };
            *reinterpret_cast<v4f*>(dst) = v0;
            *reinterpret_cast<v4f*>(dst + 16) = v1;
        }
        __syncthreads();
        if (z + 2 < z1 + 1) stash(z + 2);
        __syncthreads();
    }
}

// Layer 1 of the BF16 pass on the BF16 matrix cores with split operands: each velocity value
// v = v_h + v_l and each weight w = w_h + w_l as a BF16 pair (v_h, w_h rounded to nearest, the
// rest rounded again), and w v taken as w_h v_h + w_h v_l + w_l v_h, which is within about 2^-16
// of it, far below the BF16 rounding of the layer's output.  A slab cell holds
// (v_h0, v_h1, v_h2, v_l0, v_l1, v_l2, 0, 0); a tap takes K = 16 (two lane groups that both read
// that cell): weights (w_h, w_h, 0) against it for the first group, (w_l, 0, 0) for the second,
// so a K = 32 step covers two taps (14 steps for 27 taps, the last half empty).
constexpr int NW1S = 14 * 2 * 64;  // bf16x8 operands of the split layer 1

// wb[(s * 2 + nb) * 64 + l]: output channel 8 (l%16 / 4) + 4 nb + l%4, so that a lane ends with eight consecutive channels
// of its cell, one 16-byte store; lane group g = l/16 takes tap 2 s + g/2
__device__ __forceinline__ void wprep1_split(int k, const float* __restrict__ w, bf16x8* __restrict__ wb)
{
    const int l = k & 63, nb = (k >> 6) & 1, st = k >> 7, g = l >> 4;
    const int o = 8 * ((l & 15) >> 2) + 4 * nb + (l & 3), t = 2 * st + (g >> 1);
    bf16x8 v = bf16x8{ 0, 0, 0, 0, 0, 0, 0, 0 };
    if (t < TAPS) {
#pragma unroll
        for (int ci = 0; ci < CIO; ++ci) {
            const float x = w[(o * CIO + ci) * TAPS + t];
            const bf16 hi = (bf16)x;
            const bf16 lo = (bf16)(x - (float)hi);
            if ((g & 1) == 0) {
                v[ci] = hi;
                v[3 + ci] = hi;
            } else {
                v[ci] = lo;
            }
        }
    }
    wb[k] = v;
}

// A block works as those of the layers above, two planes a step through a ring of six slabs, one row of two planes a
// wavefront; all weights stay in registers, so that the LDS serves one read per two instructions.  G = 101: 59 us with
// the weights read from LDS (three reads per two instructions, sixteen wavefronts, two barriers a plane), now 45.
__global__ __launch_bounds__(kZThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k3c_zconv1_split(
    int32_t G, int zp, const float* __restrict__ vel, const bf16x8* __restrict__ wb, const float* __restrict__ bias,
    bf16* __restrict__ out)
{
    constexpr int NCELL = ZSY * ZSX, STEPS = 14, ITEMS = (2 * NCELL + kZThreads - 1) / kZThreads;
    static_assert(ZY == kZThreads / 64 && ZX == 32, "a row of two M-blocks per wavefront");
    __shared__ bf16x8 s_v[ZRING * NCELL];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, grp = lane >> 4;
    const int tiles_x = (G + ZX - 1) / ZX, tiles_y = (G + ZY - 1) / ZY;
    const int64_t b = blockIdx.x;
    const int tx0 = (int)(b % tiles_x) * ZX, ty0 = (int)((b / tiles_x) % tiles_y) * ZY;
    const int z0 = (int)(b / ((int64_t)tiles_x * tiles_y)) * zp;
    const int z1 = min(z0 + zp, G);
    const int64_t GG = (int64_t)G * G, n = GG * G;

    // this thread's cells of two planes: offset in a plane (from a clamped position), whether it lies in the grid
    uint32_t from[ITEMS];
    bool in[ITEMS];
    int plane[ITEMS], cell[ITEMS];
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const int e = min(tid + k * kZThreads, 2 * NCELL - 1);
        plane[k] = e >= NCELL;
        cell[k] = e;
        const int i = e - plane[k] * NCELL, gy = ty0 + i / ZSX - 1, gx = tx0 + i % ZSX - 1;
        in[k] = gy >= 0 && gy < G && gx >= 0 && gx < G;
        from[k] = (uint32_t)min(max(gy, 0), G - 1) * (uint32_t)G + (uint32_t)min(max(gx, 0), G - 1);
    }
    float pf[ITEMS][CIO];
    auto fetch = [&](int p) {  // unconditional loads: they stay in flight while a step's taps run
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            const float* at = vel + (int64_t)min(max(p + plane[k], 0), G - 1) * GG + from[k];
#pragma unroll
            for (int ci = 0; ci < CIO; ++ci) pf[k][ci] = at[ci * n];
        }
    };
    auto stash = [&](int p, int slot) {  // zero outside the grid
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            const bool on = in[k] && p + plane[k] >= 0 && p + plane[k] < G;
            bf16x8 v = bf16x8{ 0, 0, 0, 0, 0, 0, 0, 0 };
#pragma unroll
            for (int ci = 0; ci < CIO; ++ci) {
                const float x = on ? pf[k][ci] : 0.f;
                const bf16 hi = (bf16)x;
                v[ci] = hi;
                v[3 + ci] = (bf16)(x - (float)hi);
            }
            if ((k + 1) * kZThreads <= 2 * NCELL || tid + k * kZThreads < 2 * NCELL) s_v[slot * NCELL + cell[k]] = v;
        }
    };
    fetch(z0 - 1);
    stash(z0 - 1, 0);
    fetch(z0 + 1);
    stash(z0 + 1, 2);
    fetch(z0 + 3);

    bf16x8 w[STEPS][2];
#pragma unroll
    for (int st = 0; st < STEPS; ++st)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) w[st][nb] = wb[(st * 2 + nb) * 64 + lane];
    const v4f bl0 = *reinterpret_cast<const v4f*>(bias + 8 * grp), bl1 = *reinterpret_cast<const v4f*>(bias + 8 * grp + 4);
    // the lane's cell of each step's tap within a plane (past the last tap, where the weights are zero, the last again)
    int at[STEPS];
#pragma unroll
    for (int st = 0; st < STEPS; ++st) {
        const int t = min(2 * st + (grp >> 1), TAPS - 1);
        at[st] = (wave + t / 3 % 3) * ZSX + t % 3 + col;
    }
    const bool second = grp >= 2;
    const unsigned to = (tx0 + col) * C + 8 * grp;  // the lane's place in a row of the result
    __syncthreads();
    int slot = 0;  // of plane z - 1
    for (int z = z0; z < z1; z += 2) {
        const int slot2 = slot == 4 ? 0 : slot + 2, slot4 = slot == 0 ? 4 : slot - 2;
        stash(z + 3, slot4);
        fetch(z + 5);
        __builtin_amdgcn_sched_barrier(0);  // the loads stay ahead of the step's taps
        const int plane_at[4] = { slot * NCELL, (slot + 1) * NCELL, slot2 * NCELL, (slot2 + 1) * NCELL };
        v4f acc[2][2][2];  // output plane, M-block, channels
#pragma unroll
        for (int st = 0; st < STEPS; ++st)
#pragma unroll
            for (int oz = 0; oz < 2; ++oz) {
                const int d0 = 2 * st / 9, d1 = min(2 * st + 1, TAPS - 1) / 9;  // the two taps' planes
                const int base = d0 == d1 ? plane_at[oz + d0] : second ? plane_at[oz + d1] : plane_at[oz + d0];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const bf16x8 a = s_v[base + at[st] + 16 * h];
                    acc[oz][h][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[st][0], a, st == 0 ? bl0 : acc[oz][h][0], 0, 0, 0);
                    acc[oz][h][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[st][1], a, st == 0 ? bl1 : acc[oz][h][1], 0, 0, 0);
                }
            }
        auto emit = [&](int oz, int h) {
            bf16x8 v;
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = (bf16)fmaxf(acc[oz][h][k >> 2][k & 3], 0.f);
            *reinterpret_cast<bf16x8*>(out + ((int64_t)(z + oz) * GG + (int64_t)(ty0 + wave) * G) * C + to + 16 * h * C) = v;
        };
        if (ty0 + wave < G) {
            if (tx0 + ZX <= G && z + 1 < z1) {  // without a branch a block
#pragma unroll
                for (int k = 0; k < 4; ++k) emit(k >> 1, k & 1);
            } else {
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (z + (k >> 1) < z1 && tx0 + 16 * (k & 1) + col < G) emit(k >> 1, k & 1);
            }
        }
        slot = slot2;
        __syncthreads();
    }
}

// Layers 2 and 3 of the FP32 pass, 32 -> 32, on the BF16 matrix instruction with activations and weights as
// three BF16 values each (split.h), as z-sweeps.  A block owns a column of ZY x ZX cells, zp output planes and
// 16 of the 32 output channels (the grid's second dimension is the half), so that all 27 taps' weights, 81 KiB,
// fit in LDS.  It reads each input plane once, as one slab with its one-cell border, split where it enters
// LDS (so an activation is split about three times in all, not 27); the next plane is loaded into
// registers while this one is used.  An input plane p feeds output planes p + 1, p and p - 1, whose accumulators
// are kept for two 16-cell M-blocks per wavefront, the products of the high parts and the small products apart
// until the end; a tap (dy, dx) of the plane is 36 matrix instructions: three depths, two M-blocks, six products.
//
// What bounds it: matrix instructions, 324 per wavefront and plane (16.5 cycles each), and with them the 300 or
// so vector instructions of the split (3 cycles each, which add up, cnn_rows.h).
constexpr int NWS = TAPS * 2 * 3 * 64;    // bf16x8 of layers 2 and 3: half, (dy, dx), dz, part
constexpr int ZROWV = ZSY * ZSX * 4;      // bf16x8 of one part of a slab: 64 bytes a cell
constexpr int ZSCHUNKS = ZSY * ZSX * (C / 4);
constexpr int ZSCH_PER_THREAD = (ZSCHUNKS + kZThreads - 1) / kZThreads;

// ws[(((nb * 9 + t9) * 3 + dz) * 3 + part) * 64 + l][j]: that part of W[16 nb + l%16][8 (l/16) + j][dz][t9]
__device__ __forceinline__ void wprep_split(int k, const float* __restrict__ w, bf16x8* __restrict__ ws)
{
    const int l = k & 63, part = (k >> 6) % 3, dz = (k / 192) % 3, t9 = (k / 576) % 9, nb = k / 5184;
    bf16x8 v;
#pragma unroll
    for (int j = 0; j < 8; ++j)
        v[j] = split_part(w[((16 * nb + (l & 15)) * C + 8 * (l >> 4) + j) * TAPS + dz * 9 + t9], part);
    ws[k] = v;
}

// One part of a slab in LDS: four 16-byte chunks of eight channels a cell, chunk c of cell i at place
// c ^ 2 (i / 4 mod 2).  A 16-byte read is served in groups of 16 lanes (see zcell), here eight consecutive cells at
// chunk c and eight others at chunk 3 - c; eight consecutive cells take each place of a 256-byte line of four
// cells twice, i / 4 odd and even, which the exchange puts on chunks c and c ^ 2, and 3 - c has the other
// parity: no two of the sixteen share a bank.
__device__ __forceinline__ int slab_slot(int cell, int c)
{
    return cell * 4 + (c ^ ((cell >> 1) & 2));
}

__global__ __launch_bounds__(kZThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k3c_zsplit_f32(
    int32_t G, int zp, const float* __restrict__ in, const bf16x8* __restrict__ ws, const float* __restrict__ bias,
    float* __restrict__ out)
{
    constexpr int NW = NWS / 2;
    __shared__ bf16x8 s_w[NW];
    __shared__ bf16x8 s_slab[3 * ZROWV];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int col = lane & 15, grp = lane >> 4;
    const int tiles_x = (G + ZX - 1) / ZX, tiles_y = (G + ZY - 1) / ZY;
    const int64_t b = blockIdx.x;
    const int tx0 = (int)(b % tiles_x) * ZX, ty0 = (int)((b / tiles_x) % tiles_y) * ZY;
    const int z0 = (int)(b / ((int64_t)tiles_x * tiles_y)) * zp;
    const int z1 = min(z0 + zp, G);
    const int64_t GG = (int64_t)G * G;
    const int nb = blockIdx.y;

    // plane p of the slab, four channels a load, from clamped positions; what lies outside the grid is zeroed
    // when it is split into LDS (a thread past the end repeats the last chunk).  A chunk's place in the
    // plane is the same in every plane: formed once (per plane it was half of the sweep's vector instructions).
    v4f pf[ZSCH_PER_THREAD];
    unsigned at[ZSCH_PER_THREAD];
    u32x2* to[ZSCH_PER_THREAD];
    bool on[ZSCH_PER_THREAD];
#pragma unroll
    for (int k = 0; k < ZSCH_PER_THREAD; ++k) {
        const int e = min(tid + k * kZThreads, ZSCHUNKS - 1), cell = e >> 3;
        const int gy = ty0 + cell / ZSX - 1, gx = tx0 + cell % ZSX - 1;
        on[k] = gy >= 0 && gy < G && gx >= 0 && gx < G;
        at[k] = (min(max(gy, 0), G - 1) * G + min(max(gx, 0), G - 1)) * C + 4 * (e & 7);
        to[k] = reinterpret_cast<u32x2*>(s_slab + slab_slot(cell, (e & 7) >> 1)) + (e & 1);
    }
    auto fetch = [&](int p) {
        const float* plane = in + (int64_t)min(max(p, 0), G - 1) * GG * C;
#pragma unroll
        for (int k = 0; k < ZSCH_PER_THREAD; ++k) pf[k] = *reinterpret_cast<const v4f*>(plane + at[k]);
    };
    auto stash = [&](int p) {
        const bool pin = p >= 0 && p < G;
#pragma unroll
        for (int k = 0; k < ZSCH_PER_THREAD; ++k) {
            const v4f x = on[k] && pin ? pf[k] : v4f{ 0.f, 0.f, 0.f, 0.f };
            u32x2 h, m, l;
            uint32_t ph, pm, pl;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                split_pair(x[2 * j], x[2 * j + 1], ph, pm, pl);
                h[j] = ph;
                m[j] = pm;
                l[j] = pl;
            }
            to[k][0] = h;
            to[k][2 * ZROWV] = m;
            to[k][4 * ZROWV] = l;
        }
    };
    fetch(z0 - 1);
    for (int k = tid; k < NW; k += kZThreads) s_w[k] = ws[nb * NW + k];
    stash(z0 - 1);
    __syncthreads();

    const v4f zero = v4f{ 0.f, 0.f, 0.f, 0.f };
    const v4f bl = *reinterpret_cast<const v4f*>(bias + 16 * nb + 4 * grp);  // of the lane's output channels
    v4f hi[3][2], lo[3][2];  // [dz][M-block]: output planes p + 1 - dz
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            hi[d][h] = bl;
            lo[d][h] = zero;
        }
    // wavefront: cells (ty0 + wave, tx0 + 16 h + col), h = 0, 1
    for (int p = z0 - 1; p <= z1; ++p) {
        if (p < z1) fetch(p + 1);  // lands while this plane is used
        int ln = lane;
        asm volatile("" : "+v"(ln));  // the addresses are formed per plane, not held in registers
        const int cell0 = wave * ZSX + (ln & 15), q = ln >> 4;
        bf16x8 w[2][3][3], x[2][2][3];
        auto load = [&](int t9) {
#pragma unroll
            for (int d = 0; d < 3; ++d)
#pragma unroll
                for (int part = 0; part < 3; ++part) w[t9 & 1][d][part] = s_w[((t9 * 3 + d) * 3 + part) * 64 + ln];
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int part = 0; part < 3; ++part)
                    x[t9 & 1][h][part] = s_slab[part * ZROWV + slab_slot(cell0 + 16 * h + (t9 / 3) * ZSX + t9 % 3, q)];
        };
        load(0);
#pragma unroll
        for (int t9 = 0; t9 < 9; ++t9) {
            __builtin_amdgcn_sched_barrier(0);
            if (t9 + 1 < 9) load(t9 + 1);
            __builtin_amdgcn_sched_barrier(0);  // the next tap's reads are issued before this tap's products
            constexpr int wp[6] = { 2, 0, 0, 1, 1, 0 }, xp[6] = { 0, 0, 2, 1, 0, 1 };
#pragma unroll
            for (int k = 0; k < 6; ++k)
#pragma unroll
                for (int d = 0; d < 3; ++d)
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        v4f& acc = k == 1 ? hi[d][h] : lo[d][h];
                        acc = mfma_bf16(w[t9 & 1][d][wp[k]], x[t9 & 1][h][xp[k]], acc);
                    }
        }
        __builtin_amdgcn_sched_barrier(0);
        // output plane p - 1 is complete
        const int zo = p - 1, gy = ty0 + wave;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int gx = tx0 + 16 * h + col;
            if (zo >= z0 && gy < G && gx < G) {
                v4f v = hi[2][h] + lo[2][h];
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = fmaxf(v[r], 0.f);
                *reinterpret_cast<v4f*>(out + ((int64_t)zo * GG + (int64_t)gy * G + gx) * C + 16 * nb + 4 * grp) = v;
            }
#pragma unroll
            for (int d = 2; d > 0; --d) {
                hi[d][h] = hi[d - 1][h];
                lo[d][h] = lo[d - 1][h];
            }
            hi[0][h] = bl;
            lo[0][h] = zero;
        }
        if (p < z1) {
            __syncthreads();  // every wavefront is done with this plane's slab
            stash(p + 1);
            __syncthreads();
        }
    }
}

// Layer 4 of the FP32 pass (32 -> 3) as a z-sweep on the FP32 matrix instruction (a product of one weight and
// one activation is rounded once, which the split form does not do).  Rows 4 o + dz of one A block are output
// component o and kernel depth dz, so a tap (dy, dx) of an input plane is eight instructions of K = 4 per 16 cells
// for all three output planes it feeds, and a lane's result holds, for component l / 16, the three depths:
// the sums of the unfinished planes move down one element per plane.  The rest is k3c_zsplit_f32's.  On the
// vector ALUs, a cell per thread and nine sums each, the layer took 284 us at G = 128 and 77 us at G = 9.
constexpr int NW4F = 9 * 2 * 64;              // v4f of layer 4's weights: (dy, dx), half of the channels
constexpr int Z4LINES = ZSY * ZSX / 2;        // 256-byte lines of a slab, two cells each
static_assert(ZSX % 2 == 0, "a slab row starts a line");

// The chunk (four channels) that lane group q reads as half h of its eight: 2q and 2q + 1, exchanged for q >= 2,
// and chunk c's place in a slab: in a line k of two cells, cell p of it at (8 p + c + 2 k) mod 16.  Eight
// consecutive cells at one chunk and eight at another of the other parity (a 16-lane group of a 16-byte read,
// see zcell) then fall in distinct banks.
__host__ __device__ constexpr int chunk4(int q, int h)
{
    return 2 * q + (h ^ (q >> 1));
}
__device__ __forceinline__ int slab4_slot(int cell, int c)
{
    const int k = cell >> 1;
    return k * 16 + ((8 * (cell & 1) + c + 2 * k) & 15);
}

// w4f[(t9 * 2 + h) * 64 + l][j] = W4[o][4 chunk4(l/16, h) + j][dz][t9] with l%16 = 4 o + dz (zero for o = 3, dz = 3)
__device__ __forceinline__ void wprep4_f32(int k, const float* __restrict__ w, v4f* __restrict__ w4f)
{
    const int l = k & 63, h = (k >> 6) & 1, t9 = k >> 7, o = (l & 15) >> 2, dz = l & 3;
    v4f v;
#pragma unroll
    for (int j = 0; j < 4; ++j)
        v[j] = o < CIO && dz < 3 ? w[(o * C + 4 * chunk4(l >> 4, h) + j) * TAPS + dz * 9 + t9] : 0.f;
    w4f[k] = v;
}

__global__ __launch_bounds__(kZThreads) void k3c_zconv4_f32(int32_t G, int zp, const float* __restrict__ in,
                                                             const v4f* __restrict__ w4f,
                                                             const float* __restrict__ bias, float* __restrict__ disp)
{
    __shared__ v4f s_w[NW4F];
    __shared__ v4f s_slab[Z4LINES * 16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int col = lane & 15, grp = lane >> 4;
    const int tiles_x = (G + ZX - 1) / ZX, tiles_y = (G + ZY - 1) / ZY;
    const int64_t b = blockIdx.x;
    const int tx0 = (int)(b % tiles_x) * ZX, ty0 = (int)((b / tiles_x) % tiles_y) * ZY;
    const int z0 = (int)(b / ((int64_t)tiles_x * tiles_y)) * zp;
    const int z1 = min(z0 + zp, G);
    const int64_t GG = (int64_t)G * G;

    v4f pf[ZSCH_PER_THREAD];
    unsigned at[ZSCH_PER_THREAD];
    int to[ZSCH_PER_THREAD];
    bool on[ZSCH_PER_THREAD];
#pragma unroll
    for (int k = 0; k < ZSCH_PER_THREAD; ++k) {
        const int e = min(tid + k * kZThreads, ZSCHUNKS - 1), cell = e >> 3;
        const int gy = ty0 + cell / ZSX - 1, gx = tx0 + cell % ZSX - 1;
        on[k] = gy >= 0 && gy < G && gx >= 0 && gx < G;
        at[k] = (min(max(gy, 0), G - 1) * G + min(max(gx, 0), G - 1)) * C + 4 * (e & 7);
        to[k] = slab4_slot(cell, e & 7);
    }
    auto fetch = [&](int p) {
        const float* plane = in + (int64_t)min(max(p, 0), G - 1) * GG * C;
#pragma unroll
        for (int k = 0; k < ZSCH_PER_THREAD; ++k) pf[k] = *reinterpret_cast<const v4f*>(plane + at[k]);
    };
    auto stash = [&](int p) {
        const bool pin = p >= 0 && p < G;
#pragma unroll
        for (int k = 0; k < ZSCH_PER_THREAD; ++k) s_slab[to[k]] = on[k] && pin ? pf[k] : v4f{ 0.f, 0.f, 0.f, 0.f };
    };
    fetch(z0 - 1);
    for (int k = tid; k < NW4F; k += kZThreads) s_w[k] = w4f[k];
    stash(z0 - 1);
    __syncthreads();
    const float bo = grp < CIO ? bias[grp] : 0.f;
    v4f acc[2];  // per M-block: element dz is output plane p + 1 - dz
    acc[0] = acc[1] = v4f{ 0.f, 0.f, 0.f, 0.f };
    for (int p = z0 - 1; p <= z1; ++p) {
        if (p < z1) fetch(p + 1);  // lands while this plane is used
        const int cell0 = wave * ZSX + col;
#pragma unroll
        for (int t9 = 0; t9 < 9; ++t9) {
            v4f w[2], x[2][2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                w[h] = s_w[(t9 * 2 + h) * 64 + lane];
#pragma unroll
                for (int m = 0; m < 2; ++m)
                    x[m][h] = s_slab[slab4_slot(cell0 + 16 * m + (t9 / 3) * ZSX + t9 % 3, chunk4(grp, h))];
            }
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int m = 0; m < 2; ++m)
                        acc[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[h][j], x[m][h][j], acc[m], 0, 0, 0);
        }
        // output plane p - 1 is complete
        const int zo = p - 1, gy = ty0 + wave;
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const int gx = tx0 + 16 * m + col;
            if (zo >= z0 && gy < G && gx < G && grp < CIO)
                disp[grp * GG * G + (int64_t)zo * GG + (int64_t)gy * G + gx] = acc[m][2] + bo;
            acc[m] = v4f{ 0.f, acc[m][0], acc[m][1], 0.f };
        }
        if (p < z1) {
            __syncthreads();  // every wavefront is done with this plane's slab
            stash(p + 1);
            __syncthreads();
        }
    }
}

// All operand-ordered weights of a pass in one launch (each launch of them took 4.2 us, of a 44 us pass
// at G = 16).
__global__ void k3c_prep_bf16(const float* __restrict__ w1, const float* __restrict__ w2, const float* __restrict__ w3,
                              const float* __restrict__ w4, bf16x8* __restrict__ wb1, bf16x8* __restrict__ wb2,
                              bf16x8* __restrict__ wb3, bf16x8* __restrict__ wb4)
{
    int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < NWB) return wprep_bf16(k, w2, wb2);
    if ((k -= NWB) < NWB) return wprep_bf16(k, w3, wb3);
    if ((k -= NWB) < NW1S) return wprep1_split(k, w1, wb1);
    if ((k -= NW1S) < TAPS * 64) wprep4_bf16(k, w4, wb4);
}
constexpr int kPrepBf16 = 2 * NWB + NW1S + TAPS * 64;

__global__ void k3c_prep_f32(const float* __restrict__ w2, const float* __restrict__ w3, const float* __restrict__ w4,
                             bf16x8* __restrict__ ws2, bf16x8* __restrict__ ws3, v4f* __restrict__ w4f)
{
    int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < NWS) return wprep_split(k, w2, ws2);
    if ((k -= NWS) < NWS) return wprep_split(k, w3, ws3);
    if ((k -= NWS) < NW4F) wprep4_f32(k, w4, w4f);
}
constexpr int kPrepF32 = 2 * NWS + NW4F;

// Planes per block of a z-sweep over `tiles` columns, `slots` blocks running at once: the length that makes
// the busiest place's planes fewest, a block costing about three planes besides its own (its weights and the two
// planes before its first).  With 32 planes whatever the overlay, small ones ran as a handful of long
// blocks: the FP32 pass took 0.46 ms at G = 32 as at G = 64, and the BF16 pass 304 us at G = 101, whose fourth
// segment had 5 planes.
inline int z_planes(int G, int64_t tiles, int slots)
{
    int best = G;
    int64_t cost = -1;
    for (int r = 1; r <= 4; ++r) {
        int64_t segs = tiles < (int64_t)r * slots ? (int64_t)r * slots / tiles : 1;
        if (segs > G) segs = G;
        const int zp = (int)((G + segs - 1) / segs);
        segs = (G + zp - 1) / zp;
        const int64_t c = (tiles * segs + slots - 1) / slots * (zp + 3);
        if (cost < 0 || c < cost) {
            cost = c;
            best = zp;
        }
    }
    return best;
}

}  // namespace

size_t cnn3_workspace_bytes(int32_t G)
{
    const size_t cells = (size_t)G * G * G;
    return 2 * cells * C * sizeof(float) + (2 * (size_t)NWS + (size_t)NW4F) * sizeof(bf16x8);
}

void run_predict3(cnnsns_mesh3_s& m, const float* vel, const cnnsns_cnn& w, int32_t precision, float* disp,
                  hipStream_t stream)
{
    if (precision != CNNSNS_F32 && precision != CNNSNS_BF16) fail(CNNSNS_EINVAL, "predict3d: unsupported precision");
    std::lock_guard<std::mutex> lock(m.ws.mu);
    workspace_acquire(m.ws, cnn3_workspace_bytes(m.G), stream, "predict3d");
    const int32_t G = m.G;
    const int64_t cells = (int64_t)G * G * G;
    const unsigned grid = cnn_persistent_grid();
    const int64_t ztiles = (int64_t)((G + ZX - 1) / ZX) * ((G + ZY - 1) / ZY);
    int zp = z_planes(G, ztiles, (int)grid);
    if (precision == CNNSNS_BF16) zp += zp & 1;  // two planes a step
    const int64_t zblocks = ztiles * ((G + zp - 1) / zp);
    if (zblocks > (int64_t)UINT32_MAX) fail(CNNSNS_EINVAL, "predict3d: overlay too large");
    float* act0 = static_cast<float*>(m.ws.ptr);
    float* act1 = act0 + cells * C;
    bf16x8* wb2 = reinterpret_cast<bf16x8*>(act1 + cells * C);
    bf16x8* wb3 = wb2 + NWS;
    if (precision == CNNSNS_BF16) {
        bf16* b0 = reinterpret_cast<bf16*>(act0);
        bf16* b1 = reinterpret_cast<bf16*>(act1);
        bf16x8* wb1 = wb2 + NWB;  // after layer 2's operands in their region, and layer 4's after layer 3's
        bf16x8* wb4 = wb3 + NWB;
        k3c_prep_bf16<<<(kPrepBf16 + kBlock - 1) / kBlock, kBlock, 0, stream>>>(w.w[0], w.w[1], w.w[2], w.w[3], wb1, wb2,
                                                                              wb3, wb4);
        k3c_zconv1_split<<<(unsigned)zblocks, kZThreads, 0, stream>>>(G, zp, vel, wb1, w.b[0], b0);
        k3c_zsweep_bf16<2><<<(unsigned)zblocks, kZThreads, 0, stream>>>(G, zp, b0, wb2, w.b[1], b1, nullptr);
        k3c_zsweep_bf16<2><<<(unsigned)zblocks, kZThreads, 0, stream>>>(G, zp, b1, wb3, w.b[2], b0, nullptr);
        k3c_zsweep_bf16<1><<<(unsigned)zblocks, kZThreads, 0, stream>>>(G, zp, b0, wb4, w.b[3], nullptr, disp);
    } else {
        v4f* w4f = reinterpret_cast<v4f*>(wb3 + NWS);
        k3c_prep_f32<<<(kPrepF32 + kBlock - 1) / kBlock, kBlock, 0, stream>>>(w.w[1], w.w[2], w.w[3], wb2, wb3, w4f);
        k3c_zconv1<<<(unsigned)zblocks, kZ1Threads, 0, stream>>>(G, zp, vel, w.w[0], w.b[0], act0);
        const int zp2 = z_planes(G, 2 * ztiles, (int)grid);
        const dim3 g2((unsigned)(ztiles * ((G + zp2 - 1) / zp2)), 2);
        k3c_zsplit_f32<<<g2, kZThreads, 0, stream>>>(G, zp2, act0, wb2, w.b[1], act1);
        k3c_zsplit_f32<<<g2, kZThreads, 0, stream>>>(G, zp2, act1, wb3, w.b[2], act0);
        k3c_zconv4_f32<<<(unsigned)zblocks, kZThreads, 0, stream>>>(G, zp, act0, w4f, w.b[3], disp);
    }
    hip_check(hipGetLastError(), "predict3d launch");
    workspace_used(m.ws, stream);
}

}  // namespace cnnsns
