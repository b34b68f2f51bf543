// HIP kernels (gfx950) of the MRS filament path other than the pair sum.
//
//   k_pack_aos        n x 3 caller arrays -> source records
//   k_store_list      the work list of a captured evaluation
//   k_rod_forces      per segment: A = sum_j D^j_{k+1} (D^j_k)^T, its principal
//                     square root, mid frame, F and N (Sec. II.B, Eqs.
//                     mid_triad, F_comp_discrete, N_comp_discrete; Alg. 1);
//                     per node: the point force and torque on the fluid
//                     (Eqs. discrete_f, discrete_n) written straight into the
//                     pair kernel's source records
//   k_lj_boxes, k_lj_forces  Lennard-Jones repulsion between filaments (Sec. IV)
//   k_lj_rods         both and the rod forces, for few points
//   k_reduce<EPI>     fixed-order FP64 sum of the split-K partials, scaling,
//                     and the element-wise step epilogue (Eqs. newx, newD)
//   k_small_steps     whole steps of ensembles of at most 64 points
//   k_parareal_correct  Parareal correction of one slice boundary
//   k_rotsqrt         batched principal 3x3 rotation square root
//
// Source records: FP32C positions in units of eps (rho = x/eps) split
// hi + lo, forces f/eps and torques n/eps^2; FP64 records hold x, f, n.
#include <hip/hip_runtime.h>

#include <cstring>

#include "mrs_device_pairs.h"
#include "mrs_device_rod.h"
#include "mrs_internal.h"

namespace mrs {

__global__ __launch_bounds__(kBlock) void k_rotsqrt(int64_t count, const double *__restrict__ R,
                                                    double *__restrict__ S) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= count) return;
    double A[9], q[4], h[4], o[9];
    for (int k = 0; k < 9; k++) A[k] = R[9 * i + k];
    rot_to_quat(A, q);
    quat_half(q, h);
    quat_to_matrix(h, o);
    for (int k = 0; k < 9; k++) S[9 * i + k] = o[k];
}

// ------------------------------------------------------------ pack / rod

// Descriptor of source block b from the positions X (SoA, or AoS with
// aos), one wave: the same hi/lo split as the records (split_pos).
__device__ __forceinline__ void block_desc_from_x(const EnsDesc &E, const double *__restrict__ X, bool aos, int b) {
    const int N = E.N;
    const int i = b * kDescPoints + (int)(threadIdx.x & 63);
    const bool real = i < N;
    float h[3] = {0.f, 0.f, 0.f}, l[3] = {0.f, 0.f, 0.f};
    if (real) {
#pragma unroll
        for (int c = 0; c < 3; c++) split_pos(aos ? X[3 * (size_t)i + c] : X[(size_t)c * N + i], E.inv_eps, h[c], l[c]);
    }
    src_block_desc(E.wanch, E.blk, b, i, real, h[0], h[1], h[2], l[0], l[1], l[2]);
}

// One thread per point; with block descriptors (E.blk set) every wave
// (64 consecutive points, block-aligned) also writes its block's descriptor.
// The first copy_blocks blocks take the evaluation's work list, n16 16-byte
// words in mapped host memory, to the device meanwhile: without the copy
// command before it, and with two staging buffers in turn, an evaluation of
// 5,003 points (FP32C) takes 53.8 instead of 67.3 us, of 25,600 612 instead of
// 626 (one stream, MI355X).
__global__ __launch_bounds__(kBlock) void k_pack_aos(const EnsDesc E, const uint4 *__restrict__ src,
                                                     uint4 *__restrict__ dst, int n16, int copy_blocks) {
    if ((int)blockIdx.x < copy_blocks) {
        const int q = blockIdx.x * kBlock + threadIdx.x;
        if (q < n16) dst[q] = src[q];
        return;
    }
    const int i = ((int)blockIdx.x - copy_blocks) * kBlock + threadIdx.x;
    const double *X = E.Xin_aos;
    if (i < E.N) {
        if (E.form == REC_F32) reinterpret_cast<RecF32 *>(E.rec)[i] = input_rec_f32(E, i);
        else reinterpret_cast<RecF64 *>(E.rec)[i] = input_rec_f64(E, i);
    }
    const int b = i / kDescPoints;  // wave-uniform
    if (E.blk && b * kDescPoints < E.N) block_desc_from_x(E, X, true, b);
}

// The work list of a captured evaluation: a graph replays kernel arguments, while
// a copy would read the host memory again, which by then holds something else.
// 3.8 KB per launch, 20 launches at 12,800 points; eager calls copy.
__global__ __launch_bounds__(kBlock) void k_store_list(uint4 *__restrict__ dst, int n, const ListPart part) {
    const int q = threadIdx.x;
    if (q < n) dst[q] = part.v[q];
}
static_assert(kListWords <= kBlock, "one thread per word");

// One block per filament (rod_filament), or one wave per source-block
// descriptor (RodItem with fil < 0): the descriptors depend only on the
// positions, so they are written beside the filaments' records.
__global__ __launch_bounds__(kBlock) void k_rod_forces(int stage_state, int elastic, int scheme, int stage,
                                                        double dt, const EnsDesc *__restrict__ desc,
                                                       const RodItem *__restrict__ items) {
    const RodItem it = items[blockIdx.x];
    const EnsDesc E = global_desc(desc[it.ens]);
    if (it.fil < 0) {  // the whole block takes this branch
        const int b = (-1 - it.fil) * (kBlock / 64) + (int)(threadIdx.x >> 6);
        if (b * kDescPoints < E.N) block_desc_from_x(E, stage_state ? E.Xs : E.X, false, b);
        return;
    }
    const int k0 = E.off[it.fil];
    rod_filament<kBlock, false>(stage_state, elastic, scheme, stage, dt, E, k0, E.off[it.fil + 1] - k0);
}

// mrs_rod_forces_device: one block per filament on the caller's row-major
// arrays, with the descriptor and the offsets as kernel arguments.  Bound by
// latency (one chain of square roots and divisions per segment, 192 B per
// point).  The call took 150 us for 200 filaments of 128 points when it
// staged its arrays as SoA (18 strided copies of 8-byte rows, 49 us, and an
// allocation, a synchronisation and a free per call), 7 us so (MI355X).
__global__ __launch_bounds__(kBlock) void k_rod_forces_aos(const EnsDesc E, const RodOffsets off) {
    const int f = blockIdx.x;
    const int k0 = off.list ? off.list[f] : (off.step ? f * off.step : off.v[f]);
    const int k1 = off.list ? off.list[f + 1] : (off.step ? k0 + off.step : off.v[f + 1]);
    rod_filament<kBlock, true>(0, 1, 0, 0, 0.0, E, k0, k1 - k0);
}

// ------------------------------------------------------------ Lennard-Jones

__device__ __forceinline__ double wave_min_d(double v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v = fmin(v, __shfl_xor(v, off, 64));
    return v;
}

__device__ __forceinline__ double wave_max_d(double v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
    return v;
}

static_assert(kLjBlockPoints <= 64, "an LJ source block fits one wave, one point per lane");

// Value of v in lane l (l wave-uniform), read into scalar registers.
__device__ __forceinline__ double readlane_d(double v, int l) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)b, l);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Box of every LJ source block (at most kLjBlockPoints consecutive points of
// one filament) of the (stage) positions: one wave per block.
__global__ __launch_bounds__(kBlock) void k_lj_boxes(int stage_state, const EnsDesc *__restrict__ desc,
                                                     const PointItem *__restrict__ items) {
    const PointItem it = items[blockIdx.x];
    const EnsDesc E = global_desc(desc[it.ens]);
    const int b = it.p0 + (int)(threadIdx.x >> 6);
    if (b >= E.n_ljblk) return;  // wave-uniform
    const int N = E.N;
    const double *__restrict__ X = stage_state ? E.Xs : E.X;
    const int k = E.lj_blk[3 * b] + (int)(threadIdx.x & 63);
    const bool real = k < E.lj_blk[3 * b + 1];
    double lo[3], hi[3];
#pragma unroll
    for (int c = 0; c < 3; c++) {
        const double v = real ? X[(size_t)c * N + k] : 0.0;
        lo[c] = wave_min_d(real ? v : INFINITY);
        hi[c] = wave_max_d(real ? v : -INFINITY);
    }
    if ((threadIdx.x & 63) == 0) {
        double *bx = E.lj_box + 6 * (size_t)b;
#pragma unroll
        for (int c = 0; c < 3; c++) { bx[c] = lo[c]; bx[3 + c] = hi[c]; }
    }
}

// Lennard-Jones force on every point (Sec. IV): the sum over points of other
// filaments closer than r_c of 24 e (2 (sig/r)^12 - (sig/r)^6) (x_i - x_j)/r^2.
// A block owns up to 64 targets (one per lane).  Boxes first, then points:
// source blocks whose box comes within r_c of the targets are found one per
// lane, their points within r_c of the targets' box likewise, and only those
// few points are paired with the targets, by all kLjWaves waves, whose partial
// forces are added in wave order.
constexpr int kLjWaves = 8;
constexpr uint64_t kLjShare = 0x0101010101010101;  // lanes (sources) of wave 0: every kLjWaves-th
static_assert(kLjWaves == 8, "kLjShare");

struct LjConst {
    double rc2, sig2, c24;
    __device__ __forceinline__ explicit LjConst(const EnsDesc &E)
        : rc2(E.lj_rc * E.lj_rc), sig2(E.lj_sig * E.lj_sig), c24(24.0 * E.lj_e) {}
};

// r < r_c is tested as r^2 < r_c^2 and 1/r^2 is one reciprocal refined twice
// (the force vanishes at r_c = 2^(1/6) sigma, so a decision that differs from
// r < r_c by a rounding changes no force).
__device__ __forceinline__ void lj_pair(const LjConst &L, double r0, double r1, double r2, bool other, double *acc) {
    const double rr2 = fma(r2, r2, fma(r1, r1, r0 * r0));
    if (!other || !(rr2 < L.rc2)) return;
    double inv = __builtin_amdgcn_rcp(rr2);
    inv = fma(inv, fma(-rr2, inv, 1.0), inv);
    inv = fma(inv, fma(-rr2, inv, 1.0), inv);
    const double s2 = L.sig2 * inv, s6 = s2 * s2 * s2;
    const double cf = L.c24 * fma(2.0 * s6, s6, -s6) * inv;
    acc[0] = fma(cf, r0, acc[0]);
    acc[1] = fma(cf, r1, acc[1]);
    acc[2] = fma(cf, r2, acc[2]);
}

// Squared distance of the box lo, hi to the box lo1, hi1 (or point, lo1 = hi1).
__device__ __forceinline__ double lj_gap2(const double *lo, const double *hi, const double *lo1, const double *hi1) {
    double gap2 = 0.0;
#pragma unroll
    for (int c = 0; c < 3; c++) {
        const double g = fmax(0.0, fmax(lo[c] - hi1[c], lo1[c] - hi[c]));
        gap2 += g * g;
    }
    return gap2;
}

// The waves' partial forces of a block's targets, added in wave order.
__device__ __forceinline__ void lj_combine(const double (*sPart)[3][64], int lane, double *acc) {
#pragma unroll
    for (int c = 0; c < 3; c++) {
        double v = sPart[0][c][lane];
#pragma unroll
        for (int q = 1; q < kLjWaves; q++) v += sPart[q][c][lane];
        acc[c] = v;
    }
}

// General form: aligned blocks of 64 targets; also writes the LJ mask of its
// points: the FP32C pair kernels evaluate those sources in FP64, since the
// equal and opposite contact forces largely cancel at a distance and FP32
// terms would leave their rounding behind.  The source blocks are tested one
// per lane against the boxes of the targets' runs (targets of one filament; the
// last of kLjRuns boxes holds all further runs), those left against each
// target: neighbours in the order may lie far apart, so one box around all 64
// targets would leave 175 of 1,000 blocks instead of 4.  1,000 swimmers of 51
// points take 16 us, 62 when every target was tested against every block and a
// visited block's points went to one wave (MI355X).
constexpr int kLjRuns = 4;
constexpr int kLjGroups = 256;  // groups of 64 source blocks per pass

__global__ __launch_bounds__(64 * kLjWaves) void k_lj_forces(int stage_state, const EnsDesc *__restrict__ desc,
                                                             const PointItem *__restrict__ items) {
    __shared__ uint64_t sNear[kLjGroups];
    __shared__ double sRun[kLjRuns][6];
    __shared__ double sPart[kLjWaves][3][64];
    const PointItem it = items[blockIdx.x];
    const EnsDesc E = global_desc(desc[it.ens]);
    const int N = E.N;
    const double *__restrict__ X = stage_state ? E.Xs : E.X;
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint64_t share = kLjShare << w;
    const int i = it.p0 + lane;
    const bool real = i < N;
    const int ii = real ? i : N - 1;
    const double x[3] = {X[ii], X[(size_t)N + ii], X[2 * (size_t)N + ii]};
    const int fi = E.fil[ii];
    const LjConst L(E);
    double acc[3] = {0.0, 0.0, 0.0};
    const int nblk = E.n_ljblk;
    // boxes of the runs, six bounds each, shared by the waves
    const int before = __shfl_up(fi, 1, 64);  // by all lanes, or lane 1 reads from a masked one
    const uint64_t starts = __ballot(lane == 0 || fi != before ? 1 : 0);
    const int run = min(__popcll(starts & (~0ull >> (63 - lane))) - 1, kLjRuns - 1);
    const int runs = min(__popcll(starts), kLjRuns);
    for (int q = w; q < 6 * runs; q += kLjWaves) {
        const int c = q % 6;
        const double v = c % 3 == 0 ? x[0] : (c % 3 == 1 ? x[1] : x[2]);
        const double m = c < 3 ? wave_min_d(run == q / 6 ? v : INFINITY) : wave_max_d(run == q / 6 ? v : -INFINITY);
        if (lane == 0) sRun[q / 6][c] = m;
    }
    for (int b0 = 0; b0 < nblk; b0 += 64 * kLjGroups) {
        __syncthreads();
        const int groups = min(kLjGroups, (nblk - b0 + 63) / 64);
        for (int g = w; g < groups; g += kLjWaves) {
            const int bq = b0 + 64 * g + lane, b = min(bq, nblk - 1);
            const int fb = E.lj_blk[3 * b + 2];
            double bx[6];
#pragma unroll
            for (int c = 0; c < 6; c++) bx[c] = E.lj_box[6 * (size_t)b + c];
            bool close = false;
            for (int r = 0; r < runs; r++) close = close || lj_gap2(bx, bx + 3, sRun[r], sRun[r] + 3) < L.rc2;
            uint64_t mask = 0;
            for (uint64_t m = __ballot(close && bq < nblk ? 1 : 0); m; m &= m - 1) {
                const int q = __builtin_ctzll(m);
                double b1[6];
#pragma unroll
                for (int c = 0; c < 6; c++) b1[c] = readlane_d(bx[c], q);
                const int f1 = __builtin_amdgcn_readlane(fb, q);
                if (__any(real && f1 != fi && lj_gap2(b1, b1 + 3, x, x) < L.rc2 ? 1 : 0)) mask |= 1ull << q;
            }
            if (lane == 0) sNear[g] = mask;
        }
        __syncthreads();
        for (int g = 0; g < groups; g++) {
            for (uint64_t m = sNear[g]; m; m &= m - 1) {
                const int *blk = E.lj_blk + 3 * (b0 + 64 * g + __builtin_ctzll(m));
                const bool other = real && blk[2] != fi;
                // lane = source; of those within r_c of a run's box wave w
                // takes every kLjWaves-th lane, broadcast from lane registers
                const int j0 = blk[0], jn = blk[1] - j0;  // jn <= kLjBlockPoints
                double y[3];
#pragma unroll
                for (int c = 0; c < 3; c++) y[c] = X[(size_t)c * N + j0 + min(lane, jn - 1)];
                bool close = false;
                for (int r = 0; r < runs; r++) close = close || lj_gap2(y, y, sRun[r], sRun[r] + 3) < L.rc2;
                for (uint64_t src = __ballot(close && lane < jn ? 1 : 0) & share; src; src &= src - 1) {
                    const int q = __builtin_ctzll(src);
                    lj_pair(L, x[0] - readlane_d(y[0], q), x[1] - readlane_d(y[1], q), x[2] - readlane_d(y[2], q),
                            other, acc);
                }
            }
        }
    }
#pragma unroll
    for (int c = 0; c < 3; c++) sPart[w][c][lane] = acc[c];
    __syncthreads();
    if (w != 0) return;
    lj_combine(sPart, lane, acc);
    if (real) {
#pragma unroll
        for (int c = 0; c < 3; c++) E.flj[(size_t)c * N + i] = acc[c];
    }
    const bool pushed = real && (acc[0] != 0.0 || acc[1] != 0.0 || acc[2] != 0.0);
    const uint64_t mask = __ballot(pushed ? 1 : 0);
    if (lane == 0 && it.p0 < N) E.lj_mask[it.p0 / kLjMaskPoints] = mask;
}

// Repulsion and rod forces of one filament in one launch, for ensembles of at
// most kLjRodPoints points in kLjRodBlocks source blocks whose pair kernel
// reads no LJ mask: every block takes all positions into LDS and makes the
// boxes itself, so k_lj_boxes, k_lj_forces and k_rod_forces, each a chain of
// memory latencies on a nearly idle chip, become one.  Rods of at most kRodNodes
// nodes are summed out of LDS while other waves make the boxes; longer ones by
// rod_filament.  25 swimmers of 51 points take 7.9 us instead of 4.2 + 12.8 +
// 5.5 (9.6 with rod_filament after the repulsion: its loads of frames and loads
// alone took 1.9 us; MI355X).  Near the limit a block holds 120 KB of LDS, one
// block per CU, and the largest ensemble of a batch sets that for all: still
// faster than the three launches before it (their sum and this launch): 16
// ensembles of 3,162 points 47.6 and 40.6 us, one of 3,162 with 64 of 306 points
// 31.3 and 18.1, with 24 of 306 points 29.2 and 13.3 (11.8 without the large one).
__global__ __launch_bounds__(64 * kLjWaves) void k_lj_rods(int stage_state, int elastic, int scheme, int stage,
                                                           double dt, const EnsDesc *__restrict__ desc,
                                                           const RodItem *__restrict__ items) {
    extern __shared__ double sX[];  // positions, [3][N]
    __shared__ double sBox[kLjRodBlocks][6];
    __shared__ int sBlk[kLjRodBlocks][3];
    __shared__ double sPart[kLjWaves][3][64];
    constexpr int kThreads = 64 * kLjWaves, kLoads = 8;
    constexpr int kRodThreads = 128, kRodNodes = 128, kSegWaves = kRodNodes / 64;
    __shared__ double sD[9][kRodNodes];
    __shared__ double sF[3][kRodNodes + 1], sN[3][kRodNodes + 1], sdX[3][kRodNodes + 1];
    static_assert(kLjRodBlocks <= 64, "one source block per lane");
    const RodItem it = items[blockIdx.x];
    const EnsDesc E = global_desc(desc[it.ens]);
    const int N = E.N, nblk = E.n_ljblk;
    const double *__restrict__ X = stage_state ? E.Xs : E.X;
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint64_t share = kLjShare << w;
    if (it.fil < 0) {  // the whole block takes this branch (RodItem: kBlock / 64 descriptors)
        const int b = (-1 - it.fil) * (kBlock / 64) + w;
        if (w < kBlock / 64 && b * kDescPoints < N) block_desc_from_x(E, X, false, b);
        return;
    }
    const int k0 = E.off[it.fil], k1 = E.off[it.fil + 1];
    // every load the block starts from is in flight before the first is waited
    // for (each is an L2 miss: the last kernel wrote it on other XCDs)
    const int M = k1 - k0;
    const bool whole = M <= kRodNodes;  // block-uniform: the rod in one pass, out of LDS
    const bool node = whole && tid < M;
    double Dp[9], ext[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0}, clock = 0.0;
    if (w < (kRodNodes + 63) / 64) {
        const double *__restrict__ D = stage_state ? E.Ds : E.D;
        const int p = max(min(k0 + tid, k1 - 1), 0);
#pragma unroll
        for (int c = 0; c < 9; c++) Dp[c] = D[(size_t)c * N + p];
#pragma unroll
        for (int c = 0; c < 3; c++) {
            if (E.fext) ext[c] = E.fext[(size_t)c * N + p];
            if (E.next) ext[3 + c] = E.next[(size_t)c * N + p];
        }
        if (E.has_wave) clock = *E.clock;
    }
    const int blk = E.lj_blk[min(tid, 3 * nblk - 1)];
    for (int q0 = 0; q0 < 3 * N; q0 += kLoads * kThreads) {
        double v[kLoads];
#pragma unroll
        for (int u = 0; u < kLoads; u++) v[u] = X[min(q0 + u * kThreads + tid, 3 * N - 1)];
#pragma unroll
        for (int u = 0; u < kLoads; u++)
            if (q0 + u * kThreads + tid < 3 * N) sX[q0 + u * kThreads + tid] = v[u];
    }
    if (tid < 3 * nblk) sBlk[tid / 3][tid % 3] = blk;
    if (elastic < 0) elastic = E.elastic;
    if (node) {
#pragma unroll
        for (int c = 0; c < 9; c++) sD[c][tid] = Dp[c];
    }
    if (tid < 9) (tid < 3 ? sF[tid] : (tid < 6 ? sN[tid - 3] : sdX[tid - 6]))[0] = 0.0;
    __syncthreads();
    // the rod's segments by the first waves (node t: the segment after it, slot
    // t + 1), the boxes by the others, four lanes per box and coordinate
    if (w < kSegWaves) {
        if (elastic && node) {
            double F[3] = {0.0, 0.0, 0.0}, Nv[3] = {0.0, 0.0, 0.0}, dX[3] = {0.0, 0.0, 0.0};
            if (tid < M - 1)
                rod_segment<false>(E, sX, N, k0 + tid, &sD[0][0], kRodNodes, tid, (tid + 0.5) * E.ds,
                                   wave_time(E, clock, scheme, stage, dt), F, Nv, dX);
#pragma unroll
            for (int c = 0; c < 3; c++) {
                sF[c][tid + 1] = F[c];
                sN[c][tid + 1] = Nv[c];
                sdX[c][tid + 1] = dX[c];
            }
        }
    } else {
        for (int q = (tid >> 2) - 16 * kSegWaves; q < 3 * nblk; q += 16 * (kLjWaves - kSegWaves)) {
            const int b = q / 3, c = q - 3 * b, j0 = sBlk[b][0], j1 = sBlk[b][1] - 1;
            double lo = INFINITY, hi = -INFINITY;
#pragma unroll
            for (int k = 0; k < kLjBlockPoints; k += 4) {
                const double v = sX[c * N + min(j0 + k + (tid & 3), j1)];
                lo = fmin(lo, v);
                hi = fmax(hi, v);
            }
#pragma unroll
            for (int off = 1; off <= 2; off <<= 1) {
                lo = fmin(lo, __shfl_xor(lo, off, 4));
                hi = fmax(hi, __shfl_xor(hi, off, 4));
            }
            if ((tid & 3) == 0) { sBox[b][c] = lo; sBox[b][3 + c] = hi; }
        }
    }
    __syncthreads();
    const LjConst L(E);
    double lj[3] = {0.0, 0.0, 0.0};  // force on node tid (whole)
    for (int p0 = k0; p0 < k1; p0 += 64) {
        const int i = p0 + lane;
        const bool real = i < k1;
        const int ii = real ? i : k1 - 1;
        const double x[3] = {sX[ii], sX[N + ii], sX[2 * N + ii]};
        double acc[3] = {0.0, 0.0, 0.0};
        // the targets are themselves a source block: its box against the
        // others', one per lane
        const int own = __builtin_ctzll(__ballot(lane < nblk && sBlk[min(lane, nblk - 1)][0] == p0 ? 1 : 0));
        const int q = min(lane, nblk - 1);
        const bool close = lane < nblk && sBlk[q][2] != it.fil &&
                           lj_gap2(sBox[q], sBox[q] + 3, sBox[own], sBox[own] + 3) < L.rc2;
        for (uint64_t m = __ballot(close ? 1 : 0); m; m &= m - 1) {
            const int bb = __builtin_ctzll(m);
            // lane = source; of those within r_c of the targets' box wave w
            // takes every kLjWaves-th lane
            const int j0 = sBlk[bb][0], jn = sBlk[bb][1] - j0, jl = j0 + min(lane, jn - 1);
            const double y[3] = {sX[jl], sX[N + jl], sX[2 * N + jl]};
            const uint64_t in = __ballot(lane < jn && lj_gap2(y, y, sBox[own], sBox[own] + 3) < L.rc2 ? 1 : 0);
            for (uint64_t src = in & share; src; src &= src - 1) {
                const int q = __builtin_ctzll(src);
                lj_pair(L, x[0] - readlane_d(y[0], q), x[1] - readlane_d(y[1], q), x[2] - readlane_d(y[2], q), real, acc);
            }
        }
#pragma unroll
        for (int c = 0; c < 3; c++) sPart[w][c][lane] = acc[c];
        __syncthreads();
        if (w == (whole ? (p0 - k0) / 64 : 0) && real) {
            lj_combine(sPart, lane, lj);
            if (!whole) {
#pragma unroll
                for (int c = 0; c < 3; c++) E.flj[(size_t)c * N + i] = lj[c];
            }
        }
        __syncthreads();
    }
    if (!whole) {
        rod_filament<kRodThreads, false, kThreads>(stage_state, elastic, scheme, stage, dt, E, k0, M);
    } else if (node) {  // as rod_filament
        double g[3], m[3];
#pragma unroll
        for (int c = 0; c < 3; c++) { g[c] = ext[c] + lj[c]; m[c] = ext[3 + c]; }
        if (elastic) rod_node<kRodNodes + 1>(sF, sN, sdX, tid, g, m);
        store_rec(E, k0 + tid, sX[k0 + tid], sX[N + k0 + tid], sX[2 * N + k0 + tid], g[0], g[1], g[2], m[0], m[1], m[2]);
    }
}

// ------------------------------------------------------- reduce + epilogue

// One block per kReducePoints points: the waves each sum a fixed share of
// the split-K chunks for the block's points (lane = point), the parts are
// combined through LDS in wave order, and wave 0 runs the epilogue.
template <int EPI>
__global__ __launch_bounds__(kReduceThreads) void k_reduce(int stage, int scheme, double dt,
                                                   const EnsDesc *__restrict__ desc,
                                                   const PointItem *__restrict__ items) {
    __shared__ double sPart[kReduceThreads / 64][6][64];
    const PointItem it = items[blockIdx.x];
    const EnsDesc E = global_desc(desc[it.ens]);
    const int N = E.N;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int i = it.p0 + lane;
    const int K = E.K;
    const int k0 = (K * w) / (kReduceThreads / 64), k1 = (K * (w + 1)) / (kReduceThreads / 64);
    double acc[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    // wave 0 loads the state its epilogue updates before the partial sums,
    // so that the two memory latencies overlap
    double xv[3] = {0.0, 0.0, 0.0}, dv[9], uav[3] = {0.0, 0.0, 0.0}, wav[3] = {0.0, 0.0, 0.0};
    double kv[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < 9; k++) dv[k] = 0.0;
    if (EPI != EPI_WRITE && w == 0 && i < N) {
#pragma unroll
        for (int c = 0; c < 3; c++) xv[c] = E.X[(size_t)c * N + i];
#pragma unroll
        for (int k = 0; k < 9; k++) dv[k] = E.D[(size_t)k * N + i];
        if (EPI != EPI_EULER && stage > 0) {
#pragma unroll
            for (int c = 0; c < 3; c++) {
                uav[c] = E.Ua[(size_t)c * N + i];
                wav[c] = E.Wa[(size_t)c * N + i];
                if (scheme == 0) kv[c] = E.Ks[(size_t)c * N + i];
            }
        }
    }
    if (i < N) {
        const double *__restrict__ part = E.part;
        // unrolled so that several chunks' loads are in flight; the sum
        // order (k ascending) is unchanged
#pragma unroll 4
        for (int k = k0; k < k1; k++)
#pragma unroll
            for (int c = 0; c < 6; c++) acc[c] += part[((size_t)k * 6 + c) * N + i];
    }
#pragma unroll
    for (int c = 0; c < 6; c++) sPart[w][c][lane] = acc[c];
    __syncthreads();
    if (w != 0 || i >= N) return;
#pragma unroll
    for (int c = 0; c < 6; c++) {
        double v = sPart[0][c][lane];
#pragma unroll
        for (int q = 1; q < kReduceThreads / 64; q++) v += sPart[q][c][lane];
        acc[c] = v;
    }
    if (dt != dt) dt = E.dt;  // NaN: per-ensemble step size
    // the step's last epilogue advances the ensemble clock (one writer)
    if ((EPI == EPI_EULER || EPI == EPI_RK_FINAL) && i == 0 && E.clock) *E.clock += dt;
    epilogue_point<EPI>(E, N, i, acc, xv, dv, uav, wav, kv, stage, scheme, dt);
}

// ------------------------------------------------- steps of small ensembles

// Whole steps of an ensemble of at most kSmallPoints points by one workgroup,
// its state in LDS from the first stage to the last: the rod loads (a thread
// per point), the pair sum (lane = target, the waves split the sources) and the
// epilogue, with barriers where the general path has launches.  SCHEME:
// kSmallEval writes U, Omega of the state, kSmallEuler steps by Euler, 0 and 1
// by the Runge-Kutta scheme of that number.
//
// Such a step is a chain of latencies, and three launches of 3 to 4 us each
// against 1.8 us of pair arithmetic on one CU: 64 FP64 points take 4.45 instead
// of 10.6 us per Euler step, 256 such ensembles 6.4 instead of 27 us (MI355X; of
// 10,450 cycles the pairs take 5,300, rod segments and nodes 2,900, the sums and
// the update 2,150).
// At 128 points one CU has four times the pairs, a step took 10.6 instead of
// 11.2 us and a call of one step 25 instead of 23, so those go by stages.  So do 65
// to 127 points, at the time of 128 (65 points 10.6 us per step, 127 points 10.9):
// the form has one lane per target, and the one measured at 128 has two targets
// per lane, the same chain at 65.
//
// Every operation and every sum is that of k_rod_forces, k_pairs_split and
// k_reduce in the same order, so the bits are the same: small_pairs<MOD> sums
// the sources j (mod MOD) as the first levels of wave_sum_n do, and the waves'
// sums are combined as its last ones.  Sources are padded by points without
// loads at the first point, whose terms are zeros.  Eight waves, not sixteen:
// at the 128 registers of sixteen the loop spills.
template <int MOD>
__device__ __forceinline__ void small_pairs(const RecF64 *sRec, int j, double tx, double ty, double tz, double e2,
                                            double c375e2, double *acc) {
    if constexpr (MOD == kSmallPoints) {
#pragma unroll
        for (int k = 0; k < 6; k++) acc[k] = 0.0;
        const RecF64 r = sRec[j];
        pair_f64(tx, ty, tz, r.x, r.y, r.z, r.fx, r.fy, r.fz, r.nx, r.ny, r.nz, e2, c375e2, acc);
    } else {
        double o[6];
        small_pairs<2 * MOD>(sRec, j, tx, ty, tz, e2, c375e2, acc);
        small_pairs<2 * MOD>(sRec, j + MOD, tx, ty, tz, e2, c375e2, o);
#pragma unroll
        for (int k = 0; k < 6; k++) acc[k] += o[k];
    }
}

template <int SCHEME>
__global__ __launch_bounds__(kSmallThreads) void k_small_steps(int nsteps, int elastic, double dt,
                                                              const EnsDesc *__restrict__ desc) {
    constexpr int kWaves = kSmallThreads / 64, P = kSmallPoints;
    static_assert(P == 64 && kWaves <= 64 && (kWaves & (kWaves - 1)) == 0, "one lane per target, wave_sum_n's order");
    constexpr int kStateVecs = SCHEME >= 0 ? 39 : 18;
    constexpr int kStages = SCHEME == 0 ? 4 : (SCHEME == 1 ? 2 : 1);
    __shared__ double sState[kStateVecs * P];
    __shared__ RecF64 sRec[P];
    __shared__ double sF[3][P + 1], sN[3][P + 1], sX[3][P + 1];
    __shared__ double sPart[kWaves][6][P];
    __shared__ double sClock;
    const EnsDesc G0 = global_desc(desc[blockIdx.x]);
    const int N = G0.N;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    if (elastic < 0) elastic = G0.elastic;
    if (dt != dt) dt = G0.dt;
    // the descriptor with the state in LDS (SoA with stride N, as in memory)
    EnsDesc E = G0;
    double *sx = sState, *sd = sx + 3 * P, *su = sd + 9 * P, *sw = su + 3 * P;
    E.X = sx; E.D = sd; E.U = su; E.W = sw;
    if (SCHEME >= 0) {
        E.Xs = sw + 3 * P; E.Ds = E.Xs + 3 * P; E.Ua = E.Ds + 9 * P; E.Wa = E.Ua + 3 * P; E.Ks = E.Wa + 3 * P;
    }
    E.clock = &sClock;
    for (int q = tid; q < 12 * N; q += kSmallThreads) {
        if (q < 3 * N) sx[q] = G0.X[q];
        else sd[q - 3 * N] = G0.D[q - 3 * N];
    }
    // this thread's node: its place in its filament and its external loads
    const bool node = tid < N;
    int seg = 0;
    bool last = true;
    double g0[3] = {0.0, 0.0, 0.0}, m0[3] = {0.0, 0.0, 0.0};
    if (node) {
        int k0 = 0, k1 = N;
        for (int f = 0; f < G0.n_fil; f++) {
            const int a = G0.off[f], b = G0.off[f + 1];
            if (tid >= a && tid < b) { k0 = a; k1 = b; }
        }
        seg = tid - k0;
        last = tid == k1 - 1;
#pragma unroll
        for (int c = 0; c < 3; c++) {
            if (G0.fext) g0[c] = G0.fext[(size_t)c * N + tid];
            if (G0.next) m0[c] = G0.next[(size_t)c * N + tid];
        }
    }
    if (tid == 0) sClock = G0.clock ? *G0.clock : 0.0;
    if (tid < 9) (tid < 3 ? sF[tid] : (tid < 6 ? sN[tid - 3] : sX[tid - 6]))[0] = 0.0;
    const double e2 = G0.rec_eps * G0.rec_eps, c375e2 = 3.75 * e2;
    __syncthreads();
    for (int step = 0; step < nsteps; step++) {
#pragma unroll 1
        for (int st = 0; st < kStages; st++) {
            const double *X = SCHEME >= 0 && st > 0 ? E.Xs : E.X;
            const double *D = SCHEME >= 0 && st > 0 ? E.Ds : E.D;
            // rod loads -> records
            if (elastic) {
                if (node) {
                    double F[3] = {0.0, 0.0, 0.0}, Nv[3] = {0.0, 0.0, 0.0}, dX[3] = {0.0, 0.0, 0.0};
                    const double t = wave_time(E, sClock, SCHEME & 1, SCHEME >= 0 ? st : 0, dt);
                    if (!last) rod_segment<false>(E, X, N, tid, D, N, tid, (seg + 0.5) * E.ds, t, F, Nv, dX);
#pragma unroll
                    for (int c = 0; c < 3; c++) {
                        sF[c][tid + 1] = F[c];
                        sN[c][tid + 1] = Nv[c];
                        sX[c][tid + 1] = dX[c];
                    }
                }
                __syncthreads();
            }
            if (node) {
                double g[3] = {g0[0], g0[1], g0[2]}, m[3] = {m0[0], m0[1], m0[2]};
                if (elastic) rod_node<P + 1>(sF, sN, sX, tid, g, m);
                sRec[tid] = rec_f64(E, X[tid], X[N + tid], X[2 * N + tid], g[0], g[1], g[2], m[0], m[1], m[2]);
            }
            if (tid >= N && tid < P) sRec[tid] = rec_f64(E, X[0], X[N], X[2 * N], 0.0, 0.0, 0.0, 0.0, 0.0, 0.0);
            __syncthreads();
            // pair sum
            double part[6];
            const RecF64 &tgt = sRec[min(lane, N - 1)];
            small_pairs<kWaves>(sRec, w, tgt.x, tgt.y, tgt.z, e2, c375e2, part);
#pragma unroll
            for (int k = 0; k < 6; k++) sPart[w][k][lane] = part[k];
            __syncthreads();
            if (node) {
                double acc[6];
#pragma unroll
                for (int k = 0; k < 6; k++) {
                    double v[kWaves];
#pragma unroll
                    for (int q = 0; q < kWaves; q++) v[q] = sPart[q][k][tid];
#pragma unroll
                    for (int off = kWaves / 2; off >= 1; off >>= 1)
#pragma unroll
                        for (int q = 0; q < off; q++) v[q] += v[q + off];
                    acc[k] = 0.0 + v[0];  // as k_reduce, from zero
                }
                double xv[3], dv[9], uav[3] = {0.0, 0.0, 0.0}, wav[3] = {0.0, 0.0, 0.0}, kv[3] = {0.0, 0.0, 0.0};
#pragma unroll
                for (int c = 0; c < 3; c++) xv[c] = E.X[c * N + tid];
#pragma unroll
                for (int k = 0; k < 9; k++) dv[k] = E.D[k * N + tid];
                if (SCHEME >= 0 && st > 0) {
#pragma unroll
                    for (int c = 0; c < 3; c++) {
                        uav[c] = E.Ua[c * N + tid];
                        wav[c] = E.Wa[c * N + tid];
                        if (SCHEME == 0) kv[c] = E.Ks[c * N + tid];
                    }
                }
                const bool final_stage = st == kStages - 1;
                if (SCHEME != kSmallEval && final_stage && tid == 0) sClock += dt;
                if (SCHEME == kSmallEval)
                    epilogue_point<EPI_WRITE>(E, N, tid, acc, xv, dv, uav, wav, kv, 0, 0, dt);
                else if (SCHEME == kSmallEuler)
                    epilogue_point<EPI_EULER>(E, N, tid, acc, xv, dv, uav, wav, kv, 0, 0, dt);
                else if (!final_stage)
                    epilogue_point<EPI_RK_STAGE>(E, N, tid, acc, xv, dv, uav, wav, kv, st, SCHEME & 1, dt);
                else
                    epilogue_point<EPI_RK_FINAL>(E, N, tid, acc, xv, dv, uav, wav, kv, st, SCHEME & 1, dt);
            }
            __syncthreads();
        }
    }
    for (int q = tid; q < 18 * N; q += kSmallThreads) {
        if (q < 12 * N) {
            if (SCHEME == kSmallEval) continue;
            if (q < 3 * N) G0.X[q] = sx[q];
            else G0.D[q - 3 * N] = sd[q - 3 * N];
        } else if (q < 15 * N) {
            G0.U[q - 12 * N] = su[q - 12 * N];
        } else {
            G0.W[q - 15 * N] = sw[q - 15 * N];
        }
    }
    if (SCHEME != kSmallEval && tid == 0 && G0.clock) *G0.clock = sClock;
}

// ------------------------------------------------- caller arrays in and out

// State in and out of an ensemble.  The host side is pinned memory that the
// kernels access themselves, so a call is one launch: consecutive threads take
// consecutive doubles of the rows (whole PCIe bursts), the gather or scatter to
// the stored order happens in device memory.  Bound by PCIe and the host's own
// copy; against a copy per array and the transposition on the host, 12,800
// points take 78 instead of 137 us in (X, D, with the wait) and 87 instead of
// 204 us out (X, D, U, Omega), 64 points 16 instead of 53 us out (MI355X).
template <bool OUT, int W>
__device__ __forceinline__ void copy_rows(const RowArray &A, const int32_t *__restrict__ inv, int64_t N, int64_t i0,
                                          int64_t n_rows, int32_t *nonfinite) {
    const int64_t q = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t row = q / W;
    if (row >= n_rows) return;
    double *v = A.soa + (q - row * W) * N + inv[i0 + row];
    if (OUT) {
        const double x = *v;
        A.rows[q] = x;
        if (!isfinite(x)) *nonfinite = 1;
    } else {
        *v = A.rows ? A.rows[q] : 0.0;
    }
}

template <bool OUT>
__global__ __launch_bounds__(kBlock) void k_rows(const RowArrays ra, const int32_t *__restrict__ inv, int64_t N,
                                                 int64_t i0, int64_t n_rows, int32_t *nonfinite) {
    const RowArray &A = ra.a[blockIdx.y];
    if (A.w == 9) copy_rows<OUT, 9>(A, inv, N, i0, n_rows, nonfinite);
    else copy_rows<OUT, 3>(A, inv, N, i0, n_rows, nonfinite);
}

__global__ void k_set_value(double *p, double v) { *p = v; }

// ------------------------------------------------------ Parareal correction

// X = Xf + Xg - Xo and D = reorth(Df + Dg - Do) for every point (SoA state).
__global__ __launch_bounds__(kBlock) void k_parareal_correct(int N, const double *__restrict__ Xf,
                                                             const double *__restrict__ Df,
                                                             const double *__restrict__ Xg,
                                                             const double *__restrict__ Dg,
                                                             const double *__restrict__ Xo,
                                                             const double *__restrict__ Do,
                                                             double *__restrict__ X, double *__restrict__ D) {
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= N) return;
#pragma unroll
    for (int c = 0; c < 3; c++) {
        const size_t k = (size_t)c * N + i;
        X[k] = Xf[k] + Xg[k] - Xo[k];
    }
    double d[9];
#pragma unroll
    for (int c = 0; c < 9; c++) {
        const size_t k = (size_t)c * N + i;
        d[c] = Df[k] + Dg[k] - Do[k];
    }
    reorthonormalize(d);
#pragma unroll
    for (int c = 0; c < 9; c++) D[(size_t)c * N + i] = d[c];
}

// ------------------------------------------------------------ clock probe

// One wave spins until `cycles` shader-clock ticks (s_memtime) have passed,
// or `max_iter` reads, and writes the shader ticks and the constant
// reference-clock ticks (s_memrealtime) that elapsed.
__global__ __launch_bounds__(64) void k_clock_probe(int64_t cycles, int64_t max_iter, uint64_t *out) {
    const uint64_t r0 = __builtin_amdgcn_s_memrealtime();
    const uint64_t t0 = __builtin_amdgcn_s_memtime();
    uint64_t t = t0;
    for (int64_t i = 0; i < max_iter && t - t0 < (uint64_t)cycles; i++) t = __builtin_amdgcn_s_memtime();
    const uint64_t r1 = __builtin_amdgcn_s_memrealtime();
    if (threadIdx.x == 0) {
        out[0] = t - t0;
        out[1] = r1 - r0;
    }
}

hipError_t launch_clock_probe(int64_t cycles, uint64_t *out, hipStream_t s) {
    hipLaunchKernelGGL(k_clock_probe, dim3(1), dim3(64), 0, s, cycles, (int64_t)1 << 26, out);
    return hipGetLastError();
}

// --------------------------------------------------------- launch wrappers

static inline unsigned blocks_for(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

hipError_t launch_pack_aos(const EnsDesc &h_desc, const void *src, void *dst, size_t bytes, hipStream_t s) {
    if (h_desc.N == 0 || bytes % sizeof(uint4)) return h_desc.N == 0 ? hipSuccess : hipErrorInvalidValue;
    const int n16 = (int)(bytes / sizeof(uint4)), copy = (int)blocks_for(n16);
    hipLaunchKernelGGL(k_pack_aos, dim3(blocks_for(h_desc.N) + copy), dim3(kBlock), 0, s, h_desc,
                       static_cast<const uint4 *>(src), static_cast<uint4 *>(dst), n16, copy);
    return hipGetLastError();
}

hipError_t launch_store_list(const void *src, void *dst, size_t bytes, hipStream_t s) {
    if (bytes % sizeof(uint4)) return hipErrorInvalidValue;
    const size_t words = bytes / sizeof(uint4);
    hipError_t e = hipSuccess;
    for (size_t w = 0; w < words && e == hipSuccess; w += kListWords) {
        const int n = (int)(words - w < (size_t)kListWords ? words - w : (size_t)kListWords);
        ListPart part{};
        std::memcpy(part.v, static_cast<const uint4 *>(src) + w, (size_t)n * sizeof(uint4));
        hipLaunchKernelGGL(k_store_list, dim3(1), dim3(kBlock), 0, s, static_cast<uint4 *>(dst) + w, n, part);
        e = hipGetLastError();
    }
    return e;
}

hipError_t launch_rod_forces(int stage_state, int elastic, int scheme, int stage, double dt,
                             const EnsDesc *d_desc, const RodItem *d_items, int n_items, hipStream_t s) {
    if (n_items == 0) return hipSuccess;
    hipLaunchKernelGGL(k_rod_forces, dim3(n_items), dim3(kBlock), 0, s, stage_state, elastic, scheme, stage, dt,
                       d_desc, d_items);
    return hipGetLastError();
}

hipError_t launch_rod_forces_aos(const EnsDesc &h_desc, const RodOffsets &off, hipStream_t s) {
    hipLaunchKernelGGL(k_rod_forces_aos, dim3(h_desc.n_fil), dim3(kBlock), 0, s, h_desc, off);
    return hipGetLastError();
}

hipError_t launch_lj(int stage_state, const EnsDesc *d_desc, const PointItem *d_box_items, int n_box_items,
                     const PointItem *d_items, int n_items, hipStream_t s) {
    if (n_items == 0) return hipSuccess;
    hipLaunchKernelGGL(k_lj_boxes, dim3(n_box_items), dim3(kBlock), 0, s, stage_state, d_desc, d_box_items);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_lj_forces, dim3(n_items), dim3(64 * kLjWaves), 0, s, stage_state, d_desc, d_items);
    return hipGetLastError();
}

hipError_t launch_lj_rods(int stage_state, int elastic, int scheme, int stage, double dt, const EnsDesc *d_desc,
                          const RodItem *d_items, int n_items, int max_points, hipStream_t s) {
    if (n_items == 0) return hipSuccess;
    hipLaunchKernelGGL(k_lj_rods, dim3(n_items), dim3(64 * kLjWaves), (size_t)max_points * 3 * sizeof(double), s,
                       stage_state, elastic, scheme, stage, dt, d_desc, d_items);
    return hipGetLastError();
}

hipError_t launch_reduce(int epi, int stage, int scheme, double dt, const EnsDesc *d_desc,
                         const PointItem *d_items, int n_items, hipStream_t s) {
    if (n_items == 0) return hipSuccess;
    const dim3 g(n_items), b(kReduceThreads);
    switch (epi) {
        case EPI_EULER: hipLaunchKernelGGL(k_reduce<EPI_EULER>, g, b, 0, s, stage, scheme, dt, d_desc, d_items); break;
        case EPI_RK_STAGE: hipLaunchKernelGGL(k_reduce<EPI_RK_STAGE>, g, b, 0, s, stage, scheme, dt, d_desc, d_items); break;
        case EPI_RK_FINAL: hipLaunchKernelGGL(k_reduce<EPI_RK_FINAL>, g, b, 0, s, stage, scheme, dt, d_desc, d_items); break;
        default: hipLaunchKernelGGL(k_reduce<EPI_WRITE>, g, b, 0, s, stage, scheme, dt, d_desc, d_items); break;
    }
    return hipGetLastError();
}

hipError_t launch_parareal_correct(int N, const double *Xf, const double *Df, const double *Xg, const double *Dg,
                                  const double *Xo, const double *Do, double *X, double *D, hipStream_t s) {
    if (N == 0) return hipSuccess;
    hipLaunchKernelGGL(k_parareal_correct, dim3(blocks_for(N)), dim3(kBlock), 0, s, N, Xf, Df, Xg, Dg, Xo, Do, X, D);
    return hipGetLastError();
}

template <bool OUT>
static hipError_t launch_rows(const RowArrays &ra, const int32_t *inv, int64_t N, int64_t i0, int64_t n_rows,
                              int32_t *nonfinite, hipStream_t s) {
    if (n_rows == 0 || ra.count == 0) return hipSuccess;
    int w = 0;
    for (int k = 0; k < ra.count; k++) w = ra.a[k].w > w ? ra.a[k].w : w;
    hipLaunchKernelGGL(k_rows<OUT>, dim3(blocks_for(n_rows * w), ra.count), dim3(kBlock), 0, s, ra, inv, N, i0, n_rows,
                       nonfinite);
    return hipGetLastError();
}

hipError_t launch_rows_in(const RowArrays &ra, const int32_t *inv, int64_t N, int64_t i0, int64_t n_rows,
                          hipStream_t s) {
    return launch_rows<false>(ra, inv, N, i0, n_rows, nullptr, s);
}

hipError_t launch_rows_out(const RowArrays &ra, const int32_t *inv, int64_t N, int64_t i0, int64_t n_rows,
                           int32_t *nonfinite, hipStream_t s) {
    return launch_rows<true>(ra, inv, N, i0, n_rows, nonfinite, s);
}

hipError_t launch_set_value(double *p, double v, hipStream_t s) {
    hipLaunchKernelGGL(k_set_value, dim3(1), dim3(1), 0, s, p, v);
    return hipGetLastError();
}

hipError_t launch_small_steps(int scheme, int nsteps, int elastic, double dt, const EnsDesc *d_desc, int n_ens,
                              hipStream_t s) {
    const dim3 g(n_ens), b(kSmallThreads);
    switch (scheme) {
        case kSmallEval: hipLaunchKernelGGL(k_small_steps<kSmallEval>, g, b, 0, s, 1, elastic, dt, d_desc); break;
        case kSmallEuler: hipLaunchKernelGGL(k_small_steps<kSmallEuler>, g, b, 0, s, nsteps, elastic, dt, d_desc); break;
        case 0: hipLaunchKernelGGL(k_small_steps<0>, g, b, 0, s, nsteps, elastic, dt, d_desc); break;
        default: hipLaunchKernelGGL(k_small_steps<1>, g, b, 0, s, nsteps, elastic, dt, d_desc); break;
    }
    return hipGetLastError();
}

hipError_t launch_rotsqrt(int64_t count, const double *R, double *S, hipStream_t s) {
    if (count == 0) return hipSuccess;
    hipLaunchKernelGGL(k_rotsqrt, dim3(blocks_for(count)), dim3(kBlock), 0, s, count, R, S);
    return hipGetLastError();
}

}  // namespace mrs
