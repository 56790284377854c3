// The successive neighbour search (Alg. 1) for a batch of points, with the
// CNN-SNS start element of Alg. 2 selected in the same kernel.
//
// One lane walks one point.  With looked-up starts (short walks, a few long
// ones) a wavefront owns 128 points and keeps all 64 lanes busy: whenever
// lanes finish their walks, the wave hands them its next unstarted points
// (ballot + lane prefix count), so a long walk does not leave the rest of its
// wave idle (on 8M points in 16M triangles, 128 points per wavefront walk 7 %
// faster than 512 and 3.5 % faster than 256).  From given starts (long walks
// of similar length for neighbouring points) a wavefront takes 64 points, one
// per lane: 20 % faster than chunks of 512 and 7 % faster than 128, the wider
// grid hiding more of each hop's latency; and a loop of hops alone (1,089 points,
// 10 diameters: 17.8 us, 24.0 in the loop that also hands out points).  Each hop is one 64-byte gather of
// the current element's record (in large batches through LDS, launch_mode);
// the geometry is FP64 with no fused multiply-add, exactly as written.
#pragma clang fp contract(off)

#include "common.h"
#include "lds_copy.h"
#include "xcd_order.h"

namespace cnnsns {
namespace {

constexpr int kWave = 64;
constexpr int kBlock = 256;
constexpr int64_t kChunk = 128;      // points per wavefront, looked-up starts (two per lane at least)

__device__ __forceinline__ int32_t cell_of(double x, int32_t G)
{
    // floor(x G) clamped to [0, G-1]; fmax takes 0 for a NaN
    return (int32_t)fmin(fmax(floor(x * (double)G), 0.0), (double)(G - 1));
}

__device__ __forceinline__ double clamp01(double v)
{
    return v < 0.0 ? 0.0 : (v > 1.0 ? 1.0 : v);
}

// With INTERP, a finished point also gets the P1 interpolant of a nodal field at x_p in its host
// element (the step after eq. 4 of Sec. 2.1), from the barycentric numerators of the last iteration:
// out = sum_j (s_j / |S_0|) nodal[node j], summed in the element's counter-clockwise node order,
// exactly as cnnsns_interpolate computes it.
enum { kInOrder = 0, kByXcd = 1, kShared = 2 };  // how the points' blocks are taken (launch_mode)

template <int MODE, bool INTERP, int WALK>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(WALK == kShared && INTERP ? 7 : 8))) void k_locate(const ElemRec* __restrict__ rec, int64_t n_tri, int64_t n,
                                                   const double2* __restrict__ xp, const int32_t* __restrict__ start,
                                                   const double2* __restrict__ origin,
                                                   const float* __restrict__ disp,
                                                   const int32_t* __restrict__ lookup, int32_t G, int32_t max_iter,
                                                   int32_t* __restrict__ host, int32_t* __restrict__ iters,
                                                   uint8_t* __restrict__ status, const int3* __restrict__ tri,
                                                   const double2* __restrict__ nodal, double2* __restrict__ out,
                                                   XcdOrder order, double near2)
{
    const int lane = threadIdx.x & (kWave - 1);
    const unsigned block = WALK == kInOrder ? blockIdx.x : order.block(), blocks = WALK == kInOrder ? gridDim.x : order.blocks;
    if (WALK != kInOrder && block >= blocks) return;
    const int64_t wave = ((int64_t)block * kBlock + threadIdx.x) / kWave;
    const int64_t n_waves = (int64_t)blocks * (kBlock / kWave);
    // From the element before movement (long paths, where neighbouring points share elements)
    // a wave takes kWave consecutive points, a lane one of them.
    // From a looked-up start (short paths, whose rare long ones cluster at the two ends of the
    // point order, the domain boundary) a wave owns kChunk slots, R = kChunk / 64 runs of 64
    // consecutive points strided across all points, so the long walks of one region spread over
    // many waves: run u is 64-point block b + u n_waves with b = wave for even u and
    // n_waves - 1 - wave for odd u, so both ends of the point order fall to the first waves,
    // which walk them first (runs in the order 0, R - 1, 1, R - 2, ...).
    auto point_of = [&](int64_t v) -> int64_t {
        const int k = (int)(v >> 6);
        const int u = (k & 1) ? (int)(kChunk / 64) - 1 - (k >> 1) : (k >> 1);
        const int64_t b = (u & 1) ? n_waves - 1 - wave : wave;
        return ((b + u * n_waves) << 6) + (v & (kWave - 1));
    };
    int64_t next = 0;  // wave-uniform: next unstarted slot
    const int64_t n_slots = kChunk;
    if (MODE == START_GIVEN && wave * kWave >= n) return;

    // Start elements that depend on a lookup (CNN-SNS, ASG) are computed for the whole chunk
    // first, eight independent load chains per lane, and kept in LDS: a lane that takes a new
    // point then waits for one load (x_p) instead of a chain of three.
    __shared__ int32_t s_start[MODE == START_GIVEN ? 1 : kBlock / kWave][MODE == START_GIVEN ? 1 : kChunk];
    int32_t* const my_start = s_start[MODE == START_GIVEN ? 0 : (threadIdx.x / kWave)];
    // Results of the lookup-started modes, whose lanes take new points as they finish, wait in LDS until
    // the wave's chunk is done and are then written run by run, 64 consecutive points at a time (the
    // start slot of a point is reused for its host).  From given starts a lane keeps its one point's
    // results in registers and writes them when the whole wave is done.
    constexpr int kStage = MODE == START_GIVEN ? 1 : kBlock / kWave;
    constexpr int kSlots = MODE == START_GIVEN ? 1 : kChunk;
    __shared__ int32_t s_iters[kStage][kSlots];
    __shared__ uint8_t s_status[kStage][kSlots];
    // with INTERP, the barycentric coordinates of x_p in the host: the interpolant is formed after the
    // loop, for all of the wave's points at once, instead of a chain of dependent gathers per finishing lane
    __shared__ double s_lam[INTERP ? kStage : 1][3][INTERP ? kSlots : 1];
    const int wslot = MODE == START_GIVEN ? 0 : (int)(threadIdx.x / kWave);
    if (MODE != START_GIVEN) {
        // in two halves of four points per lane, staged so that the four chains' loads of each
        // level issue together (eight at once would cost occupancy)
        constexpr int PER_LANE = (int)(kChunk / kWave), H = PER_LANE / 2;
        static_assert(H >= 1 && PER_LANE == 2 * H, "looked-up starts need an even number (>= 2) of points per lane");
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            int64_t pt[H];
            double2 o[H];
            int32_t k0[H];
#pragma unroll
            for (int u = 0; u < H; ++u) {
                const int64_t i = point_of((half * H + u) * kWave + lane);
                pt[u] = i < n ? i : n - 1;  // slots past the last point repeat it
                o[u] = MODE == START_CNN ? origin[pt[u]] : xp[pt[u]];
            }
            if (MODE == START_CNN) {
                float dx[H], dy[H];
#pragma unroll
                for (int u = 0; u < H; ++u) {
                    const int64_t c = (int64_t)cell_of(o[u].y, G) * G + cell_of(o[u].x, G);
                    dx[u] = disp[c];
                    dy[u] = disp[(int64_t)G * G + c];
                }
#pragma unroll
                for (int u = 0; u < H; ++u) {
                    // predicted departure point of the origin's cell (Alg. 2)
                    o[u].x = clamp01(o[u].x + (double)dx[u]);
                    o[u].y = clamp01(o[u].y + (double)dy[u]);
                }
            }
#pragma unroll
            for (int u = 0; u < H; ++u) k0[u] = lookup[(int64_t)cell_of(o[u].y, G) * G + cell_of(o[u].x, G)];
#pragma unroll
            for (int u = 0; u < H; ++u) {
                if (k0[u] < 0) k0[u] = (MODE == START_CNN && start) ? start[pt[u]] : 0;  // uncovered cell
                my_start[(half * H + u) * kWave + lane] = k0[u];
            }
        }
        __builtin_amdgcn_wave_barrier();  // LDS operations of one wavefront complete in order
    }

    // kShared: records by way of LDS.  In copy k of four, the four lanes of each quad fetch the record of their lane k,
    // 16 bytes each: the wavefront's records, quad by quad, a copy's 65 16-byte places after the one before (so that lanes
    // reading the same quarter of their records use distinct banks).
    constexpr bool SHARED = WALK == kShared;
    constexpr int kCopy = 65 * 16;
    __shared__ __attribute__((aligned(16))) char s_rec[SHARED ? kBlock / kWave : 1][SHARED ? 4 * kCopy : 16];
    char* const my_rec = s_rec[SHARED ? threadIdx.x / kWave : 0];

    bool active = false;
    int64_t idx = 0;
    int64_t slot = 0;  // the lane's current slot (lookup-started modes)
    double px = 0.0, py = 0.0;
    int32_t K = 0, I = 0;
    int fin_given = -1;          // given starts: the lane's outcome, written after the loop
    double lam_given[3] = { 0.0, 0.0, 0.0 };

    // One hop, from the record of element K at `r`: the outcome where the walk ends, else -1.
    auto hop = [&](const void* r) -> int {
        I = I + 1;
        const double2* r2 = static_cast<const double2*>(r);
        const double2 A = r2[0], B = r2[1], C = r2[2];
        const int4 nb = static_cast<const int4*>(r)[3];
        // barycentric numerators s_j = |S_j| (Sec. 2.2), vertex j's column replaced by x_p
        const double adx = A.x - px, ady = A.y - py;
        const double bdx = B.x - px, bdy = B.y - py;
        const double cdx = C.x - px, cdy = C.y - py;
        const double s0 = bdx * cdy - bdy * cdx;
        const double s1 = cdx * ady - cdy * adx;
        const double s2 = adx * bdy - ady * bdx;
        // the neighbour ids arrive with the coordinates (one 64-byte line): keep their load beside
        // the others, not sunk behind the containment test as a second dependent access
        asm volatile("" : : "v"(nb.x), "v"(nb.y), "v"(nb.z));
        int fin = -1;
        if (s0 >= 0.0 && s1 >= 0.0 && s2 >= 0.0) {
            fin = CNNSNS_FOUND;  // closed containment: all coordinates >= 0
        } else {
            // eq. (5): smallest coordinate, ties to the lowest index
            int32_t m = nb.x;
            double smin = s0;
            if (s1 < smin) { smin = s1; m = nb.y; }
            if (s2 < smin) { m = nb.z; }
            if (m == -1) {
                fin = CNNSNS_OUTSIDE;
            } else {
                K = m;
                if (I >= max_iter) fin = CNNSNS_MAXITER;
            }
        }
        if (fin >= 0) {
            double lam[3] = { 0.0, 0.0, 0.0 };
            if (INTERP) {  // barycentric coordinates s_j / |S_0| of x_p in the host
                double2 a = A, b = B, c = C;
                double t0 = s0, t1 = s1, t2 = s2;
                if (fin == CNNSNS_MAXITER) {  // the host is the element just moved to
                    const double2* q2 = reinterpret_cast<const double2*>(rec + K);
                    a = q2[0];
                    b = q2[1];
                    c = q2[2];
                    const double ax_ = a.x - px, ay_ = a.y - py, bx_ = b.x - px, by_ = b.y - py;
                    const double cx_ = c.x - px, cy_ = c.y - py;
                    t0 = bx_ * cy_ - by_ * cx_;
                    t1 = cx_ * ay_ - cy_ * ax_;
                    t2 = ax_ * by_ - ay_ * bx_;
                }
                const double area2 = (b.x - a.x) * (c.y - a.y) - (b.y - a.y) * (c.x - a.x);
                lam[0] = t0 / area2;
                lam[1] = t1 / area2;
                lam[2] = t2 / area2;
            }
            if (MODE == START_GIVEN) {
                fin_given = fin;
                if (INTERP)
                    for (int j = 0; j < 3; ++j) lam_given[j] = lam[j];
            } else {
                my_start[slot] = K;
                s_iters[wslot][slot] = I;
                s_status[wslot][slot] = (uint8_t)fin;
                if (INTERP)
                    for (int j = 0; j < 3; ++j) s_lam[wslot][j][slot] = lam[j];
            }
        }
        return fin;
    };
    if constexpr (MODE == START_GIVEN) {  // a lane walks one point
        idx = wave * kWave + lane;
        if (idx < n) {
            const double2 p = xp[idx];
            px = p.x;
            py = p.y;
            K = start[idx];
            active = K >= 0 && K < n_tri;
            if (!active) {
                fin_given = CNNSNS_BADSTART;
                K = -1;
            }
        }
        // by way of LDS where the wavefront's points lie in order: most of the 60 lanes with one before them near that one
        if (SHARED && __popcll(__ballot(idx < n && near_lane_before(near2, px, py))) >= 40) {
            const char* quarter = reinterpret_cast<const char*>(rec) + 16 * (lane & 3);
            const char* const r = my_rec + (lane & 3) * kCopy + (lane >> 2) * (int)sizeof(ElemRec);
            while (__ballot(active) != 0) {
                const int at = active ? K : 0;
                auto copy = [&](int e, int k) { lds_copy16(quarter + (int64_t)e * (int64_t)sizeof(ElemRec), my_rec + k * kCopy); };
                copy(__builtin_amdgcn_mov_dpp(at, 0x00, 0xf, 0xf, true), 0);  // lane 0 of each quad to all four
                copy(__builtin_amdgcn_mov_dpp(at, 0x55, 0xf, 0xf, true), 1);
                copy(__builtin_amdgcn_mov_dpp(at, 0xaa, 0xf, 0xf, true), 2);
                copy(__builtin_amdgcn_mov_dpp(at, 0xff, 0xf, 0xf, true), 3);
                lds_copies_arrived();
                if (active && hop(r) >= 0) active = false;
            }
        }
        while (active)
            if (hop(rec + K) >= 0) active = false;
    } else {
        for (;;) {
            // hand unstarted points of the chunk to idle lanes
            const uint64_t idle = __ballot(!active);
            if (idle != 0 && next < n_slots) {
                const uint32_t lo = (uint32_t)idle, hi = (uint32_t)(idle >> 32);
                const int rank = (int)__builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u));
                if (!active && next + rank < n_slots) {
                    const int64_t v = next + rank;
                    idx = point_of(v);
                    slot = v;
                    if (idx < n) {
                        const double2 p = xp[idx];
                        px = p.x;
                        py = p.y;
                        K = my_start[v];
                        I = 0;
                        if (K < 0 || K >= n_tri) {  // no element: host -1, path 0 (and a NaN interpolant)
                            my_start[v] = -1;
                            s_iters[wslot][v] = 0;
                            s_status[wslot][v] = CNNSNS_BADSTART;
                        } else {
                            active = true;
                        }
                    }
                }
                next += __popcll(idle);
            }
            if (__ballot(active) == 0) {
                if (next >= n_slots) break;
                continue;
            }
            if (active && hop(rec + K) >= 0) active = false;
        }
    }
    // the interpolant at x_p: sum_j lambda_j nodal[node j] over the host's nodes in counter-clockwise
    // order, NaN where there is no host
    auto interpolant = [&](int32_t k, const double (&l)[3]) -> double2 {
        if (k < 0) return double2{ __builtin_nan(""), __builtin_nan("") };
        const int3 v = tri[k];
        const double2 u0 = nodal[v.x], u1 = nodal[v.y], u2 = nodal[v.z];
        return double2{ l[0] * u0.x + l[1] * u1.x + l[2] * u2.x, l[0] * u0.y + l[1] * u1.y + l[2] * u2.y };
    };
    // the wave's results, coalesced
    if (MODE == START_GIVEN) {
        if (idx < n) {
            host[idx] = K;
            if (iters) iters[idx] = I;
            if (status) status[idx] = (uint8_t)fin_given;
            if (INTERP) out[idx] = interpolant(K, lam_given);
        }
    } else {
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int r = 0; r < (int)(kChunk / kWave); ++r) {
            const int64_t v = r * kWave + lane, i = point_of(v);
            if (i < n) {
                const int32_t k = my_start[v];
                host[i] = k;
                if (iters) iters[i] = s_iters[wslot][v];
                if (status) status[i] = s_status[wslot][v];
                if (INTERP) {
                    const double l[3] = { s_lam[wslot][0][v], s_lam[wslot][1][v], s_lam[wslot][2][v] };
                    out[i] = interpolant(k, l);
                }
            }
        }
    }
}

// P1 interpolation at x_p in its host element (the approximation that follows
// eq. 4 in Sec. 2.1): the element's nodal basis functions are its barycentric
// coordinates (Sec. 2.2), lambda_j = s_j / |S_0| with s_j the numerators the
// walk uses and |S_0| the doubled area, and the value is sum_j lambda_j u(n_j)
// over the element's nodes, summed in node order.  One thread per point;
// FP64, no fused multiply-add.
__global__ __launch_bounds__(kBlock) void k_interp(const ElemRec* __restrict__ rec, const int3* __restrict__ tri,
                                                   int64_t n_tri, int64_t n, const double2* __restrict__ xp,
                                                   const int32_t* __restrict__ host, const double2* __restrict__ nodal,
                                                   double2* __restrict__ out)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    const int32_t K = host[i];
    if (K < 0 || K >= n_tri) {  // no element (a start outside the mesh)
        out[i] = double2{ __builtin_nan(""), __builtin_nan("") };
        return;
    }
    const double2* r2 = reinterpret_cast<const double2*>(rec + K);
    const double2 A = r2[0], B = r2[1], C = r2[2], p = xp[i];
    const double adx = A.x - p.x, ady = A.y - p.y;
    const double bdx = B.x - p.x, bdy = B.y - p.y;
    const double cdx = C.x - p.x, cdy = C.y - p.y;
    const double s0 = bdx * cdy - bdy * cdx;
    const double s1 = cdx * ady - cdy * adx;
    const double s2 = adx * bdy - ady * bdx;
    const double area2 = (B.x - A.x) * (C.y - A.y) - (B.y - A.y) * (C.x - A.x);
    const double l0 = s0 / area2, l1 = s1 / area2, l2 = s2 / area2;
    const int3 v = tri[K];
    const double2 u0 = nodal[v.x], u1 = nodal[v.y], u2 = nodal[v.z];
    out[i] = double2{ l0 * u0.x + l1 * u1.x + l2 * u2.x, l0 * u0.y + l1 * u1.y + l2 * u2.y };
}

}  // namespace

void launch_interp(const cnnsns_mesh_s& m, int64_t n, const double* xp, const int32_t* host, const double* nodal,
                   double* out, hipStream_t stream)
{
    if (n == 0) return;
    const int64_t blocks = (n + kBlock - 1) / kBlock;
    if (blocks > (int64_t)INT32_MAX) fail(CNNSNS_EINVAL, "interpolate: too many points");
    k_interp<<<(unsigned)blocks, kBlock, 0, stream>>>(m.rec, reinterpret_cast<const int3*>(m.tri), m.n_tri, n,
                                                       reinterpret_cast<const double2*>(xp), host,
                                                       reinterpret_cast<const double2*>(nodal),
                                                       reinterpret_cast<double2*>(out));
    hip_check(hipGetLastError(), "interpolate launch");
}

// In order of id up to 64 blocks, by XCD from there, and from given starts with 10 wavefronts a compute unit or more (of
// 256) in the form that takes records through LDS where a wavefront's points lie in order.  There the L1 bounds
// the walk: it looks up one line a cycle, 256 a hop for 64 records of four 16-byte loads, where four lanes that fetch a
// record together need 64.  With fewer wavefronts a hop's latency counts, which the LDS adds to.  Walks of every node (n
// points), 20 diameters, in us, in order, by XCD and through LDS:
//     n      16k    20k    66k    125k   160k   250k   503k   1M     4M     8M
//     order  35.3   36.1   55.5   66.4   87.3   124    217    383    1528   3085
//     XCD    35.2   34.8   49.5   54.4   77.4   113    175    357    1511   2996
//     LDS    35.3   52.0   52.3   60.3   71.7   89     154    298    1223   2569
// (8M points, 160 diameters, whose paths have left their neighbours: 19.0, 18.9 and 19.7 ms.)  Points in no order share
// nothing that the LDS could save: 503k points, 10 diameters, 168 us with every record from memory, 187 with all through
// LDS, 165 with the wavefront's choice (in order: 130, 90 and 87).
// Looked-up starts, CNN then overlay, 20 diameters, in us, in order and by XCD: 503k points 20.2 and 17.8, 18.3 and 15.9;
// 1M 36.7 and 32.7, 32.4 and 28.6; 2.1M 97.9 and 97.6, 71.6 and 69.5.  They go in order again past 6,144 blocks, where
// their short walks have little left to share: 3.4M (6,592 blocks) 92.2 and 90.2, 77.7 and 74.2; 4M 165 and 166, 136
// and 138; 8M 310 and 310, 270 and 270; 8M in no order 678 and 679, 389 and 392.
constexpr int64_t kSharedWaves = 2560;
constexpr unsigned kOrderedBlocks = 6144;

template <int MODE, bool INTERP>
static void launch_mode(const cnnsns_mesh_s& m, int64_t n, const double2* xp2, const int32_t* start,
                        const double2* or2, const float* disp, int32_t max_iter, int32_t* host, int32_t* iters,
                        uint8_t* status, const double* nodal, double* out, unsigned blocks, hipStream_t stream)
{
    const XcdOrder order(MODE == START_GIVEN || blocks <= kOrderedBlocks ? blocks : 0, MODE == START_GIVEN ? 128 : 32);
    const double near2 = 256.0 * m.mean_diam * m.mean_diam;  // 16 diameters
    auto run = [&](auto kernel) {
        kernel<<<order.chunk ? order.grid() : blocks, kBlock, 0, stream>>>(m.rec, m.n_tri, n, xp2, start, or2, disp, m.lookup, m.G, max_iter, host,
                                                    iters, status, reinterpret_cast<const int3*>(m.tri),
                                                    reinterpret_cast<const double2*>(nodal), reinterpret_cast<double2*>(out),
                                                    order, near2);
    };
    if (order.chunk == 0)
        run(k_locate<MODE, INTERP, kInOrder>);
    else if (MODE != START_GIVEN || (int64_t)blocks * (kBlock / kWave) < kSharedWaves)
        run(k_locate<MODE, INTERP, kByXcd>);
    else
        run(k_locate<START_GIVEN, INTERP, kShared>);
}

void launch_locate(const cnnsns_mesh_s& m, int64_t n, const double* xp, const int32_t* start, const double* origin,
                   const float* disp, int32_t max_iter, int32_t* host, int32_t* iters, uint8_t* status,
                   hipStream_t stream, const double* nodal, double* out)
{
    if (n == 0) return;
    if (max_iter <= 0) max_iter = 1 << 20;
    const int64_t chunk = (!disp && start) ? kWave : kChunk;
    const int64_t waves = (n + chunk - 1) / chunk;
    const int64_t blocks = (waves * kWave + kBlock - 1) / kBlock;
    if (blocks > (int64_t)INT32_MAX) fail(CNNSNS_EINVAL, "locate: too many points");
    const auto* xp2 = reinterpret_cast<const double2*>(xp);
    const auto* or2 = reinterpret_cast<const double2*>(origin);
    const unsigned g = (unsigned)blocks;
    const bool interp = nodal != nullptr;
    if (disp) {
        if (interp)
            launch_mode<START_CNN, true>(m, n, xp2, start, or2, disp, max_iter, host, iters, status, nodal, out, g, stream);
        else
            launch_mode<START_CNN, false>(m, n, xp2, start, or2, disp, max_iter, host, iters, status, nodal, out, g, stream);
    } else if (start) {
        if (interp)
            launch_mode<START_GIVEN, true>(m, n, xp2, start, or2, disp, max_iter, host, iters, status, nodal, out, g, stream);
        else
            launch_mode<START_GIVEN, false>(m, n, xp2, start, or2, disp, max_iter, host, iters, status, nodal, out, g, stream);
    } else {
        if (interp)
            launch_mode<START_ASG, true>(m, n, xp2, start, or2, disp, max_iter, host, iters, status, nodal, out, g, stream);
        else
            launch_mode<START_ASG, false>(m, n, xp2, start, or2, disp, max_iter, host, iters, status, nodal, out, g, stream);
    }
    hip_check(hipGetLastError(), "locate launch");
}

}  // namespace cnnsns
