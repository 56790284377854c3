// The reduced-precision 2D forward passes (3x3 convolutions 2 -> 32 -> 32 -> 32 -> 2, zero "same" padding, ReLU between
// layers) as one pipeline over rows, for operands of eight K values a lane (BF16 or FP8).
//
// All four layers run in one kernel that walks down column strips of 128 pixels (122 output columns), two rows a step
// and one barrier a step: each layer works one row pair behind the rows its input needs, the rows between them live in
// LDS (three pairs of conv1's and conv2's output), and only the columns at a strip's sides and the first rows of a
// block's segment are computed twice.  Four wavefronts run conv1 and conv2, four conv3 and conv4, one of each on a
// SIMD, every one with its layers' weights in registers.
//
// One matrix instruction of K = 32 takes a tap of 32 channels.  With weights as its row operand a lane ends with eight
// channels of one pixel, in the order in which the next layer takes them: one store, and conv3's result goes into
// conv4's instruction without leaving the registers.  conv1 (K = 18) is padded to one K = 32 step, its K ordered
// tap-major so that a lane's operand is four (u, v) pairs read from LDS; conv4 (N = 2) computes, per conv3 pixel, its 18
// (output channel, tap) contributions into LDS, and the next step sums the 9 taps of every output pixel.
//
// What bounds it: matrix instructions, 160 per SIMD and step, 2,640 cycles of about 3,900; the rest is the two
// wavefronts' turns at operand reads, ReLU and barrier.  Against 14 x 30 tiles with their halo recomputed in every layer
// (38% more matrix instructions, five barriers a tile), repeated calls of the whole pass in us, before and now, in BF16:
// G = 64: 19.0 and 17.2, 256: 19.1 and 18.9, 512: 32.8 and 25.6, 1024: 81 and 48, 4096: 933 and 483; in FP8: 64: 34.8
// and 20.1, 256: 37.7 and 22.1, 512: 56 and 29, 1024: 110 and 53, 4096: 1082 and 520.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

namespace cnnsns {
namespace strips {

typedef float v4f __attribute__((ext_vector_type(4)));
constexpr int kThreads = 512;      // 8 wavefronts: 0-3 run conv1 and conv2, 4-7 conv3 and conv4, one of each a SIMD
constexpr int C = 32;
constexpr int CW = 128;            // columns of a strip in every layer, 32 a wavefront
constexpr int OW = CW - 6;         // its output columns: columns 3 .. 124
constexpr int VW = CW + 2;         // velocity columns
constexpr int AW = CW + 2;         // pixels of an activation row in LDS: one more on each side (never valid)
constexpr int ZPX = 24;            // floats of a pixel's conv4 contributions: [dx][o][dy, padded to 4]
constexpr int ZROW = CW * ZPX;
// Floats between velocity rows: conv1's lanes read pixels of up to three rows at once, which 16 banks keep apart.
constexpr int VPITCH = 144;

// Hidden activations are stored pair-interleaved: position 2c + h of a pixel holds channel c + 16 h.  With weights
// as the matrix instruction's row operand and pixels as its column operand, lane (i, q) ends with channels 4q .. 4q + 3
// and 16 + 4q .. 19 + 4q of pixel i, which are positions 8q .. 8q + 7: one store, and as they stand the
// column operand of the next instruction on that pixel.
__device__ __forceinline__ int chan_at(int pos)
{
    return (pos >> 1) + 16 * (pos & 1);
}

// packed weights, one row operand per lane:
//   w1 [nb][lane]: k = 8 (l/16) + j = 2 tap + ci (< 18, else 0) of output channel 16 nb + l%16
//   w2, w3 [tap][nb][lane]: input channel chan_at(8 (l/16) + j), output channel 16 nb + l%16
//   w4 [nb][lane]: input channel chan_at(8 (l/16) + j), row n = 16 nb + l%16 of tap and output channel as below
constexpr int P1 = 2 * 64, P2 = 9 * 2 * 64, P4 = 2 * 64;
constexpr int PACKED = P1 + 2 * P2 + P4;

// conv4's row n = 8 dx + 4 o + dy: tap (dy, dx) of output channel o; false where dx or dy is 3 (a row of zeros)
__device__ __forceinline__ bool conv4_row(int n, int& o, int& tap)
{
    const int dx = n >> 3, dy = n & 3;
    o = (n >> 2) & 1;
    tap = 3 * dy + dx;
    return dx < 3 && dy < 3;
}

// 16-byte place of chunk c of pixel p in a row of conv4's contributions: the exchange puts the eight
// pixels that a store takes at a time on distinct banks of 32.
__device__ __forceinline__ int zslot(int p, int c)
{
    return p * (ZPX / 4) + (c ^ ((p >> 2) & 1));
}

// A block's output rows: the `per` consecutive rows from linear row u of the strips laid end to end, cut at a strip's
// end; with `segs` set, block s instead takes rows [s % segs * per, + per) of strip s / segs.
struct Plan {
    int G, per, segs, blocks;
    __device__ void range(int s, int& u0, int& u1) const
    {
        if (segs) {
            u0 = s / segs * G + s % segs * per;
            u1 = min(u0 + per, (s / segs + 1) * G);
        } else {
            u0 = s * per;
            u1 = min(u0 + per, (G + OW - 1) / OW * G);
        }
    }
};

// One block per compute unit.  Whole segments of a strip, or, where the strips' count leaves too many units without a
// segment, the strips end to end: a block that meets a strip's end starts its pipeline again, about four steps of two
// rows.
inline Plan strip_rows(int G, int cus)
{
    auto cdiv = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
    const int strips = (int)cdiv(G, OW), segs = cus / strips;
    auto even = [&](int64_t a, int64_t b) { return (int)((cdiv(a, b) + 1) / 2 * 2); };
    const int per = even((int64_t)strips * G, cus);
    if (segs) {
        const int rows = even(G, segs);
        if (rows / 2 + 4 <= per / 2 + 8) {
            const int n = (int)cdiv(G, rows);
            return Plan{ G, rows, n, strips * n };
        }
    }
    return Plan{ G, per, 0, (int)cdiv((int64_t)strips * G, per) };
}

// The pass in the form F:
//   Op, mfma: the operand of eight values and its instruction; BYTES = 4 of them, a pixel's 32 channels;
//   place(p): chunk c of pixel p of an activation row sits at place c ^ place(p);
//   F(args, first, q, o): the constants of a lane of conv1 and conv2 (first) or of conv3 and conv4;
//   vel(u, v): the velocity pair as operand values;
//   start[l], act<l>(lo, hi, v): the initial accumulators of the lane's first (l = 0: conv1) and second layer and the
//     result's values, ReLU applied, as the next layer's operand words;
//   sum0, sum(s): initial value of the nine tap products' sum, and the displacement.
template <class F>
__device__ __forceinline__ void pass(int32_t G, const Plan& plan, const float* __restrict__ vel,
                                     const typename F::Op* __restrict__ packed, const typename F::Args& args,
                                     float* __restrict__ disp)
{
    using Op = typename F::Op;
    constexpr int NW = sizeof(Op) / 4;        // words of an operand
    constexpr int ROWB = AW * F::BYTES;       // bytes of an activation row
    constexpr int RING = 3 * 2 * ROWB;        // three row pairs
    constexpr int MB = 16 * F::BYTES;         // bytes between blocks of 16 columns
    struct alignas(sizeof(Op)) Words {
        uint32_t w[NW];
    };
    __shared__ __attribute__((aligned(16))) char s_act[2 * RING];  // conv1's and conv2's output rows
    __shared__ v4f s_zs[2 * 2 * ZROW / 4 + 32];                    // conv4's contributions of a row pair, twice
    v4f(*s_z)[2 * ZROW / 4] = reinterpret_cast<v4f(*)[2 * ZROW / 4]>(s_zs);
    // (u, v) as packed BF16 pairs: three row pairs and the first of them again, so that any two that follow each other
    // are four consecutive rows
    __shared__ uint32_t s_vel[8 * VPITCH];

    const int per = gridDim.x / 8, s = (blockIdx.x % 8) * per + blockIdx.x / 8;
    if (s >= plan.blocks) return;
    const int lane = threadIdx.x & 63, i = lane & 15, q = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wc = wave & 3;
    const bool first = wave < 4;  // conv1 and conv2
    const int64_t GG = (int64_t)G * G;

    Op w[9][2], wx[2];  // the 32 -> 32 layer's weights and conv1's or conv4's, in registers throughout
    {
        const Op* from = packed + P1 + (first ? 0 : P2) + lane;
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            w[t][0] = from[2 * t * 64];
            w[t][1] = from[(2 * t + 1) * 64];
        }
        from = packed + (first ? 0 : P1 + 2 * P2) + lane;
        wx[0] = from[0];
        wx[1] = from[64];
    }
    // this lane's operand reads: pixel column 32 wc + i - 1 + dx (the next 16 columns: MB bytes on); dx = 1 also its stores
    int rd[3];
#pragma unroll
    for (int dx = 0; dx < 3; ++dx) rd[dx] = (32 * wc + i + dx) * F::BYTES + (q ^ F::place(32 * wc + i + dx)) * (int)sizeof(Op);
    // conv1's operand: taps 4q + jj in the velocity window; past tap 8 the weights are zero and the first tap is read again
    int tap[4];
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
        const int t = 4 * q + jj;
        tap[jj] = 32 * wc + i + (t < 9 ? t / 3 * VPITCH + t % 3 : 0);
    }
    const int oc = 32 * wc + (lane & 31), oo = lane >> 5;  // conv4's sums: column and output channel
    const F f(args, first, q, oo);
    // lanes without a chunk of the second block (q >= 2) store it beside the rows
    int zrd[3], zwr[2], zw1[2];
    const int zr1 = q < 2 ? 1 : 0;
#pragma unroll
    for (int dx = 0; dx < 3; ++dx) zrd[dx] = zslot(min(max(oc, 1), CW - 2) - 1 + dx, 2 * dx + oo);
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) zwr[nb] = zslot(32 * wc + i, 4 * nb + q);
#pragma unroll
    for (int m = 0; m < 2; ++m) zw1[m] = q < 2 ? zwr[1] + m * 16 * (ZPX / 4) : 4 * ZROW / 4 + (lane & 31);

    auto strips = [&](auto role) {
        constexpr bool first = decltype(role)::value;  // conv1 and conv2
        int u0, u1;
        plan.range(s, u0, u1);
        while (u0 < u1) {
            const int strip = u0 / G, y0 = u0 - strip * G, n = min(u1 - u0, G - y0), x0 = strip * OW;
            u0 += n;
            const int J = (n + 3) / 2;   // row pairs of conv3
            const int yb = y0 - 3;       // conv1's first row
            const bool inner = x0 >= 3 && x0 - 3 + CW <= G;  // every column lies in the grid
            uint32_t in[2];                                  // this lane's pixel columns do
#pragma unroll
            for (int m = 0; m < 2; ++m) in[m] = (unsigned)(x0 - 3 + 32 * wc + 16 * m + i) < (unsigned)G ? ~0u : 0u;

            // Velocity rows y, y + 1: wavefronts 0, 1 and 2, 3 a row each, 64 columns a wavefront; columns 128 and 129 by the
            // second of the two (the other lanes' second values go to the row's padding).  Loaded unconditionally from
            // clamped positions, zeroed outside the grid when stashed.
            const int va = 64 * (wc & 1) + lane, vb = 128 + (lane & 1);
            const bool in_a = (unsigned)(x0 - 4 + va) < (unsigned)G, in_b = x0 - 4 + vb < G;
            const unsigned ga = 4u * min(max(x0 - 4 + va, 0), G - 1), gb = 4u * min(x0 - 4 + vb, G - 1);
            const int la = va + (wc >> 1) * VPITCH, lb = ((wc & 1) && lane < 2 ? vb : VW + lane % (VPITCH - VW)) + (wc >> 1) * VPITCH;
            float pu[2], pv[2];
            auto load = [&](const float* row) {
                const char *u = reinterpret_cast<const char*>(row), *v = reinterpret_cast<const char*>(row + GG);
                pu[0] = *reinterpret_cast<const float*>(u + ga);
                pv[0] = *reinterpret_cast<const float*>(v + ga);
                pu[1] = *reinterpret_cast<const float*>(u + gb);
                pv[1] = *reinterpret_cast<const float*>(v + gb);
            };
            auto fetch = [&](int y) { load(vel + (int64_t)min(max(y + (wc >> 1), 0), G - 1) * G); };
            auto stash = [&](const float (&pu)[2], const float (&pv)[2], bool row_in, int slot) {
                uint32_t* to = s_vel + 2 * slot * VPITCH;
                uint32_t* also = slot ? to : to + 6 * VPITCH;
                const uint32_t a = f.vel(in_a && row_in ? pu[0] : 0.f, in_a && row_in ? pv[0] : 0.f);
                const uint32_t b = f.vel(in_b && row_in ? pu[1] : 0.f, in_b && row_in ? pv[1] : 0.f);
                to[la] = a;
                to[lb] = b;
                also[la] = a;
                also[lb] = b;
            };
            auto row_in = [&](int y) { return (unsigned)y < (unsigned)G; };

            if (first) {
                float u[2][2], v[2][2];  // the first two pairs: one wait for memory
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    fetch(yb - 1 + 2 * k);
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        u[k][j] = pu[j];
                        v[k][j] = pv[j];
                    }
                }
                fetch(yb + 3);
#pragma unroll
                for (int k = 0; k < 2; ++k) stash(u[k], v[k], row_in(yb - 1 + 2 * k + (wc >> 1)), k);
            }
            const bool out_col = oc >= 3 && oc < 3 + OW && x0 - 3 + oc < G;
            float p1 = f.sum0, p2 = f.sum0;
            const float* ahead = nullptr;  // the steady steps' next velocity row and output row
            float* out = nullptr;
            __syncthreads();
            // Step t: conv1's pair t (rows yb + 2t, + 1), conv2's pair t - 2 (rows yb + 1 + 2 (t - 2), + 1), conv3's pair
            // t - 4 (rows yb + 2 + 2 (t - 4), + 1), the sums of conv3's pair t - 5.  A steady step has all of them, and all
            // its rows lie in the grid: it has no branch.  (A taken branch costs a wavefront some 40 cycles.)
            int sl = 0;  // t mod 3
            auto step = [&](int t, auto steady_, auto inner_) {
                constexpr bool steady = decltype(steady_)::value, masked = !decltype(inner_)::value;
                const int sl1 = sl == 2 ? 0 : sl + 1, sl2 = sl == 0 ? 2 : sl - 1;  // slots of pairs t - 2 (t + 1) and t - 1
                // A row's pixels (d[block of 16 columns][channels]) as the next layer's operands, zero outside the grid
                auto act = [&](auto layer, const v4f (&d)[2][2], int y, Words (&v)[2]) {
                    const uint32_t keep = steady || row_in(y) ? ~0u : 0u;
#pragma unroll
                    for (int m = 0; m < 2; ++m) {
                        f.template act<decltype(layer)::value>(d[m][0], d[m][1], v[m].w);
#pragma unroll
                        for (int k = 0; k < NW; ++k) {
                            if (masked) v[m].w[k] &= in[m];
                            if (!steady) v[m].w[k] &= keep;
                        }
                    }
                };
                auto store = [&](char* to, const Words (&v)[2]) {
#pragma unroll
                    for (int m = 0; m < 2; ++m) *reinterpret_cast<Words*>(to + rd[1] + m * MB) = v[m];
                };
                if (!first && (steady || t >= 5)) {
                    v4f z[2][3];  // conv4's contributions of the previous step
#pragma unroll
                    for (int k = 0; k < 6; ++k) z[k / 3][k % 3] = s_z[(t - 1) & 1][zrd[k % 3] + k / 3 * (ZROW / 4)];
                    // an output row's taps in the order (dy, dx), those of its first two rows carried in registers
                    const int y = yb + 1 + 2 * (t - 5);  // the first of the two output rows that are complete
                    float o[2];
#pragma unroll
                    for (int r = 0; r < 2; ++r) {
                        o[r] = f.sum(((p2 + z[r][0][2]) + z[r][1][2]) + z[r][2][2]);
                        p2 = ((p1 + z[r][0][1]) + z[r][1][1]) + z[r][2][1];
                        p1 = ((f.sum0 + z[r][0][0]) + z[r][1][0]) + z[r][2][0];
                    }
                    if (steady) {
                        if (out_col) {
                            out[0] = o[0];
                            out[G] = o[1];
                        }
                        out += 2 * G;
                    } else if (out_col && y >= y0) {
                        float* to = disp + oo * GG + (int64_t)y * G + x0 - 3 + oc;
                        to[0] = o[0];
                        if (y + 1 < y0 + n) to[G] = o[1];
                    }
                }
                constexpr int lag = first ? 2 : 4;
                if (steady || (t >= lag && t < J + (first ? 3 : 4))) {
                    // conv2's or conv3's pair: its input pairs are in slots `sl1` and `sl2` of the layer's ring (conv2's
                    // output pair k goes to slot (k + 2) mod 3 = t mod 3)
                    const char* lo = s_act + (first ? 0 : RING) + sl1 * 2 * ROWB;
                    const char* hi = s_act + (first ? 0 : RING) + sl2 * 2 * ROWB;
                    v4f acc[2][2][2];  // output row, block of 16 columns, channels
                    const int y = first ? yb + 1 + 2 * (t - 2) : yb + 2 + 2 * (t - 4);
                    auto emit = [&](int r) {
                        Words v[2];
                        act(std::integral_constant<int, 1>{}, acc[r], y + r, v);
                        if (first) {
                            store(s_act + RING + (2 * sl + r) * ROWB, v);
                        } else {
                            v4f* to = s_z[t & 1] + r * (ZROW / 4);
                            v4f c[2][2];
#pragma unroll
                            for (int k = 0; k < 4; ++k)
                                c[k >> 1][k & 1] = F::mfma(wx[k & 1], __builtin_bit_cast(Op, v[k >> 1]), v4f{ 0.f, 0.f, 0.f, 0.f });
#pragma unroll
                            for (int m = 0; m < 2; ++m) {
                                to[zwr[0] + m * 16 * (ZPX / 4)] = c[m][0];
                                s_zs[zw1[m] + zr1 * ((t & 1) * (2 * ZROW / 4) + r * (ZROW / 4))] = c[m][1];
                            }
                        }
                    };
                    constexpr int PF = 3;
                    Op x[PF + 1][2];
                    auto read = [&](int g) {
                        const char* from = (g < 6 ? lo : hi) + rd[g % 3] + (g / 3 & 1) * ROWB;
                        x[g % (PF + 1)][0] = *reinterpret_cast<const Op*>(from);
                        x[g % (PF + 1)][1] = *reinterpret_cast<const Op*>(from + MB);
                    };
#pragma unroll
                    for (int g = 0; g < PF; ++g) read(g);
#pragma unroll
                    for (int g = 0; g < 12; ++g) {  // input row g / 3, tap column g % 3
                        if (g + PF < 12) read(g + PF);
                        __builtin_amdgcn_sched_barrier(0);  // the reads stay ahead of the instructions
#pragma unroll
                        for (int r = 0; r < 2; ++r) {
                            const int dy = g / 3 - r;
                            if (dy < 0 || dy > 2) continue;
#pragma unroll
                            for (int m = 0; m < 2; ++m)
#pragma unroll
                                for (int nb = 0; nb < 2; ++nb)
                                    acc[r][m][nb] = F::mfma(w[3 * dy + g % 3][nb], x[g % (PF + 1)][m],
                                                        dy == 0 && g % 3 == 0 ? f.start[1][nb] : acc[r][m][nb]);
                        }
                        if (g == 8) emit(0);  // the first row is complete
                    }
                    emit(1);
                }
                if (first) {
                    stash(pu, pv, steady || row_in(yb + 3 + 2 * t + (wc >> 1)), sl2);
                    if (steady) {
                        load(ahead);
                        ahead += 2 * G;
                    } else {
                        fetch(yb + 5 + 2 * t);
                    }
                    if (steady || t < J + 2) {
                        v4f d[2][2][2];
                        const uint32_t* from = s_vel + 2 * sl * VPITCH;
#pragma unroll
                        for (int r = 0; r < 2; ++r)
#pragma unroll
                            for (int m = 0; m < 2; ++m) {
                                uint32_t v[4];
#pragma unroll
                                for (int jj = 0; jj < 4; ++jj) v[jj] = from[tap[jj] + r * VPITCH + 16 * m];
                                const Op x = F::gather(v);
#pragma unroll
                                for (int nb = 0; nb < 2; ++nb)
                                    d[r][m][nb] = F::mfma(wx[nb], x, f.start[0][nb]);
                            }
#pragma unroll
                        for (int r = 0; r < 2; ++r) {
                            Words v[2];
                            act(std::integral_constant<int, 0>{}, d[r], yb + 2 * t + r, v);
                            store(s_act + (2 * sl + r) * ROWB, v);
                        }
                    }
                }
                sl = sl1;
                __syncthreads();
            };
            const int steady_end = min(J + 2, (G - 5 - yb) >> 1);
            for (int t = 0; t < J + 5; ++t) {
                if (t == 6 && steady_end > 6) {
                    ahead = vel + (int64_t)(yb + 17 + (wc >> 1)) * G;
                    out = disp + oo * GG + (int64_t)y0 * G + x0 - 3 + oc;
                    if (inner)
                        for (; t < steady_end; ++t) step(t, std::true_type{}, std::true_type{});
                    else
                        for (; t < steady_end; ++t) step(t, std::true_type{}, std::false_type{});
                }
                step(t, std::false_type{}, std::false_type{});
            }
        }
    };
    if (first)
        strips(std::true_type{});
    else
        strips(std::false_type{});
}

}  // namespace strips
}  // namespace cnnsns
