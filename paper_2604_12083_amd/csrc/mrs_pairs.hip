// HIP kernels (gfx950) of the all-pairs MRS sum (Sec. II.C, Eqs.
// velocity_field, angular_velocity_field, superposition).
//
//   k_pairs_tile_*    one lane per target (T targets per lane), sources
//                     staged through LDS and broadcast to the wave, split-K
//                     over source chunks
//   k_pairs_split     small-ensemble form: a wave owns a few targets, its lanes
//                     stride over the sources and the sums are combined with
//                     wave shuffles
//   k_eval_direct     the same for a small one-shot evaluation, from the
//                     caller's arrays to the velocities in one launch
//
// Kernel functions.  With R^2 = r^2 + eps^2, Q = 1/R and H_i the kernel
// functions of the blob phi_eps (Sec. II.C), 8 pi H_i are
//   H1: Q + eps^2 Q^3            H2: Q^3
//   H3: Q^3 + 1.5 eps^2 Q^5      H4: 3.75 eps^4 Q^7 - 0.75 eps^2 Q^5 - 0.5 Q^3
//   H5: 1.5 Q^5 + 3.75 eps^2 Q^7
// The FP32C form works in units of eps (rho = r/eps, f~ = f/eps,
// n~ = n/eps^2), where the same expressions hold with eps = 1 and
// U = sum/(8 pi mu), Omega = sum/(8 pi mu eps); this keeps every FP32
// intermediate far from overflow and folds all constants into one FP64
// scale per target.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "mrs_device_pairs.h"
#include "mrs_device_rod.h"
#include "mrs_internal.h"

namespace mrs {

// ----------------------------------------------------------------- pairs

// Squared distance between the boxes [lo0, hi0] and [lo1, hi1] (0 if they overlap).
__device__ __forceinline__ float box_gap2(const float *lo0, const float *hi0, const float *lo1, const float *hi1) {
    float d2 = 0.0f;
#pragma unroll
    for (int c = 0; c < 3; c++) {
        const float g = fmaxf(0.0f, fmaxf(lo0[c] - hi1[c], lo1[c] - hi0[c]));
        d2 = fmaf(g, g, d2);
    }
    return d2;
}

// A wave whose target box is farther than this (squared, in units of eps)
// from a source block's box has no near pair in it (rho >= 4).  The boxes
// are the widened hi-part boxes of the block descriptors (src_block_desc),
// which contain the exact positions at any distance from the origin.
constexpr float kFarBoxGap2 = 17.0f;

// Anchored far blocks.  Relative to the centre c of a 64-source block's box,
// a source sits at w = (sh - c) + sl (stored with the block descriptors) and
// a target at u = (th - c) + tl, and r = u - w costs 3 instead of 9
// operations.  Each of u and w takes two FP32 roundings (at most 2^-24 of
// its magnitude each), and r one more; with the gap between the boxes larger
// than the block's half-diagonal, |w| < |r| and |u| < 2 |r|, so r keeps a
// relative error below 7 x 2^-24 < 2^-21, against 2^-23 for the exact hi/lo
// difference of the other paths.  (A gap of 4 half-diagonals, |w| <= |r|/4,
// sent more blocks down the exact-separation path and was 2.6% slower on
// 1,000 swimmers of 51 points, 3.4% on 16 batched 3,200-point slices;
// MI355X, interleaved A/B, 12,800 points even.)
constexpr float kAnchorGapRatio2 = 1.0f;

// Block descriptors and contact masks are written before the pair launch and
// only read by it, so the kernel reads them through the constant address
// space: the loads are wave-uniform and go through the scalar cache into
// scalar registers.
typedef __attribute__((address_space(4))) const float desc_float;
typedef __attribute__((address_space(4))) const uint64_t mask_word;
__device__ __forceinline__ const desc_float *desc_at(const float *blk, int64_t b) {
    return (const desc_float *)(blk + (size_t)kDescFloats * b);
}

// Persistent schedule.  The grid holds as many blocks as the device keeps
// resident; each block claims the next item of the work list from a counter
// (queue[0], an ordinary vector atomic from one lane) until the list is
// exhausted, so blocks that run ahead take more items and the device stays
// full until the last items, which the work list makes the shortest.  Every
// item still writes its own partial slot: results do not depend on which
// block ran which item.  The last block to leave (queue[1] counts them)
// resets both counters, so the next launch (or graph replay) starts at zero.
__device__ __forceinline__ int claim_item(uint32_t *queue, int *sNext) {
    __syncthreads();  // the previous item is finished and sNext has been read
    if (threadIdx.x == 0) *sNext = (int)atomicAdd(queue, 1u);
    __syncthreads();
    return *sNext;
}

__device__ __forceinline__ void leave_queue(uint32_t *queue) {
    if (threadIdx.x == 0) {
        __threadfence();
        if (atomicAdd(queue + 1, 1u) == gridDim.x - 1) {
            atomicExch(queue, 0u);
            atomicExch(queue + 1, 0u);
        }
    }
}

// Orders a wave's own LDS writes before its later reads (and its reads
// before later writes) without waiting for the other waves of the block.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The record of source i (wave-uniform), in scalar registers.
struct ScalarRec {
    float v[12];
};

__device__ __forceinline__ ScalarRec scalar_rec(const RecF32 *rec, int i) {
    const desc_float *p = (const desc_float *)(rec + __builtin_amdgcn_readfirstlane(i));
    ScalarRec r;
#pragma unroll
    for (int k = 0; k < 12; k++) r.v[k] = p[k];
    return r;
}

// Sources of one staged round, as the pair loops read them (a wave reads one
// source at a time, as broadcasts).  w is the anchored position, m = 1.5 w x n
// and k = w x f the source's parts of the split cross products (far_block),
// h + l the position in units of eps.
template <int SLOTS>
struct SrcStage {
    float4 W[SLOTS];   // w, fx
    float4 F[SLOTS];   // fy, fz, nx, ny
    float4 M[SLOTS];   // nz, m
    float4 K[SLOTS];   // k, lx
    float4 H[SLOTS];   // h, ly
    float lz[SLOTS];
    // Stages source i of E at slot j; absent (i < 0): zero loads at the anchor
    // and the origin.  A source with contact forces enters the FP32 sums with
    // zero loads; the FP64 pass evaluates it with its own loads.
    __device__ __forceinline__ void put(const EnsDesc &E, int j, int i) {
        float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b = a, c = a, w = a;
        if (i >= 0) {
            const RecF32 r = reinterpret_cast<const RecF32 *>(E.rec)[i];
            a = r.a; b = r.b; c = r.c;
            w = E.wanch[i];
            if (E.lj_mask && ((E.lj_mask[i / kLjMaskPoints] >> (i % kLjMaskPoints)) & 1)) {
                a.w = 0.0f; b.w = 0.0f;
                c = make_float4(0.f, 0.f, 0.f, 0.f);
            }
        }
        const float fx = a.w, fy = b.w, fz = c.x, nx = c.y, ny = c.z, nz = c.w;
        W[j] = make_float4(w.x, w.y, w.z, fx);
        F[j] = make_float4(fy, fz, nx, ny);
        // |w| < |r| in the blocks that use them: m and k overflow no earlier
        // (up to their factor) than the products n . r and f . r
        M[j] = make_float4(nz, 1.5f * fmaf(w.y, nz, -(w.z * ny)), 1.5f * fmaf(w.z, nx, -(w.x * nz)),
                           1.5f * fmaf(w.x, ny, -(w.y * nx)));
        K[j] = make_float4(fmaf(w.y, fz, -(w.z * fy)), fmaf(w.z, fx, -(w.x * fz)), fmaf(w.x, fy, -(w.y * fx)), b.x);
        H[j] = make_float4(a.x, a.y, a.z, b.y);
        lz[j] = b.z;
    }
};

// Sums of the staged sources [sb, se) (of one block, an even number) into p,
// for targets at u relative to the block's anchor (no near pair in the block).
//
// The loop is bound by VALU issue (the launch issues one instruction per 2.4
// clocks and SIMD, its instruction mix allows one per 2.35) and by the clock
// the card holds under it, so it is written for the fewest instructions per
// pair:
//   * The cross products are split along r = u - w: sum H3 (n x r) =
//     (sum H3 n) x u + sum H3 (w x n), and the same for f, so a pair adds
//     H3 n, H3 f and H3 m, H3 k with products m, k that the staging forms
//     once per source, and u enters once per block.
//   * H4 = u7 - H3/2 with u7 = 3.75 Q^7: its second part is -1/2 of the sum
//     H3 n already kept.  REMOTE: u7 is below half an ulp of H3/2, and H4 n
//     needs no sum of its own.
//   * H3, H5 and u7 are kept divided by 1.5 (one product less); m is staged
//     times 1.5 and the sums of H3 and of Omega are multiplied once per block.
// 42 instructions per pair and one v_rsq_f32 (REMOTE; 46 otherwise) against
// 51 for the direct form: pair kernel 58.1 -> 52.6 ms at 256,000 points, 165
// -> 151.5 us at 12,800 (one target per lane, MI355X).  Two sources at a time
// with their reciprocal roots together: 0.7% faster than one at a time at
// 256,000 points, 2% at 51,000 (swimmers); four at a time spills.
template <int T, bool REMOTE, class STAGE>
__device__ __forceinline__ void far_block(const STAGE &S, int sb, int se, const float (&ux)[T], const float (&uy)[T],
                                          const float (&uz)[T], float (&p)[T][6]) {
    constexpr int G = 2;
    float sn[T][3], sf[T][3], o[T][3];
#pragma unroll
    for (int t = 0; t < T; t++)
#pragma unroll
        for (int k = 0; k < 3; k++) { sn[t][k] = 0.0f; sf[t][k] = 0.0f; o[t][k] = 0.0f; }
#pragma unroll 2
    for (int j0 = sb; j0 < se; j0 += G) {
        float rx[G][T], ry[G][T], rz[G][T], q[G][T], fx[G];
#pragma unroll
        for (int g = 0; g < G; g++) {
            const float4 W = S.W[j0 + g];
            fx[g] = W.w;
#pragma unroll
            for (int t = 0; t < T; t++) {
                const float x = ux[t] - W.x, y = uy[t] - W.y, z = uz[t] - W.z;
                rx[g][t] = x; ry[g][t] = y; rz[g][t] = z;
                q[g][t] = rsq_f32(fmaf(z, z, fmaf(y, y, fmaf(x, x, 1.0f))));
            }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int g = 0; g < G; g++) {
            const float4 F = S.F[j0 + g], M = S.M[j0 + g], K = S.K[j0 + g];
#pragma unroll
            for (int t = 0; t < T; t++) {
                const float x = q[g][t] * q[g][t], q3 = q[g][t] * x, q5 = q3 * x;
                const float h1 = q[g][t] + q3;
                const float h3 = fmaf(2.0f / 3.0f, q3, q5);  // H3 / 1.5
                const float q7 = q5 * x;
                const float h5 = fmaf(2.5f, q7, q5);         // H5 / 1.5
                const float fr = fmaf(F.y, rz[g][t], fmaf(F.x, ry[g][t], fx[g] * rx[g][t]));
                const float nr = fmaf(M.x, rz[g][t], fmaf(F.w, ry[g][t], F.z * rx[g][t]));
                const float a = q3 * fr, b = h5 * nr;
                p[t][0] = fmaf(h3, M.y, fmaf(a, rx[g][t], fmaf(h1, fx[g], p[t][0])));
                p[t][1] = fmaf(h3, M.z, fmaf(a, ry[g][t], fmaf(h1, F.x, p[t][1])));
                p[t][2] = fmaf(h3, M.w, fmaf(a, rz[g][t], fmaf(h1, F.y, p[t][2])));
                o[t][0] = fmaf(h3, K.x, fmaf(b, rx[g][t], o[t][0]));
                o[t][1] = fmaf(h3, K.y, fmaf(b, ry[g][t], o[t][1]));
                o[t][2] = fmaf(h3, K.z, fmaf(b, rz[g][t], o[t][2]));
                sn[t][0] = fmaf(h3, F.z, sn[t][0]);
                sn[t][1] = fmaf(h3, F.w, sn[t][1]);
                sn[t][2] = fmaf(h3, M.x, sn[t][2]);
                sf[t][0] = fmaf(h3, fx[g], sf[t][0]);
                sf[t][1] = fmaf(h3, F.x, sf[t][1]);
                sf[t][2] = fmaf(h3, F.y, sf[t][2]);
                if (!REMOTE) {
                    const float u7 = 2.5f * q7;  // 3.75 Q^7 / 1.5
                    o[t][0] = fmaf(u7, F.z, o[t][0]);
                    o[t][1] = fmaf(u7, F.w, o[t][1]);
                    o[t][2] = fmaf(u7, M.x, o[t][2]);
                }
            }
        }
    }
#pragma unroll
    for (int t = 0; t < T; t++) {
        p[t][0] = fmaf(1.5f, fmaf(sn[t][1], uz[t], -(sn[t][2] * uy[t])), p[t][0]);
        p[t][1] = fmaf(1.5f, fmaf(sn[t][2], ux[t], -(sn[t][0] * uz[t])), p[t][1]);
        p[t][2] = fmaf(1.5f, fmaf(sn[t][0], uy[t], -(sn[t][1] * ux[t])), p[t][2]);
        o[t][0] = fmaf(-0.5f, sn[t][0], o[t][0] + fmaf(sf[t][1], uz[t], -(sf[t][2] * uy[t])));
        o[t][1] = fmaf(-0.5f, sn[t][1], o[t][1] + fmaf(sf[t][2], ux[t], -(sf[t][0] * uz[t])));
        o[t][2] = fmaf(-0.5f, sn[t][2], o[t][2] + fmaf(sf[t][0], uy[t], -(sf[t][1] * ux[t])));
#pragma unroll
        for (int k = 0; k < 3; k++) p[t][3 + k] = fmaf(1.5f, o[t][k], p[t][3 + k]);
    }
}

// Beyond this squared gap between the boxes u7 = 3.75 Q^7 is less than 2^-25
// of H3/2 >= Q^3/2 (7.5 Q^4 < 7.5 / 16384^2 < 2^-25), which is below half an
// ulp of any FP32 value: H4 = u7 - H3/2 rounds to -H3/2.
constexpr float kRemoteBoxGap2 = 16384.0f;

// Blocks per CU the register budget must allow: 5 with one target per lane
// (<= 102 VGPRs; four were even), 3 with two (<= 170).  PERSIST: items claimed
// from the queue; otherwise block b runs item b.
//
// QUAD (one target per lane): the block's four waves share the item's 64
// targets and split its sources, wave w taking the 64-source blocks w, w + 4,
// ... of the item; each wave stages and uses only its own blocks (no block
// barrier in the loop), and the four waves' sums are added in wave order at
// the end of the item.  A wave's share of an item is a quarter of the
// item's pairs, so the waves that run last on a SIMD hold short work.
template <int T, bool PERSIST, bool QUAD>
__global__ __launch_bounds__(kBlock, T == 1 ? 5 : 3) void k_pairs_tile_f32(const EnsDesc *__restrict__ desc,
                                                           const PairItem *__restrict__ items, int n_items,
                                                           uint32_t *queue) {
    static_assert(!QUAD || T == 1, "four-wave source split: one target per lane");
    __shared__ SrcStage<kSrcTile> S;
    static_assert(kSrcTile / kKahanBlock == kBlock / 64 && kKahanBlock == kDescPoints,
                  "one source block (one descriptor) per wave");
    __shared__ int sNext;
    int idx = PERSIST ? claim_item(queue, &sNext) : (int)blockIdx.x;
    while (idx < n_items) {
    const PairItem it = items[idx];
    const EnsDesc &E = desc[it.ens];  // not global_desc: even in time, and 12 B of spills when persistent
    const RecF32 *__restrict__ rec = reinterpret_cast<const RecF32 *>(E.rec);
    const int tid = threadIdx.x;
    // target slot of this lane: the block's lanes (tiled) or the wave's (QUAD)
    const int tl = QUAD ? (tid & 63) : tid;
    float thx[T], thy[T], thz[T], tlx[T], tly[T], tlz[T];
    float s[T][6], c[T][6];
    double pn[T][6];  // FP64 sums of the near pairs and contact sources
    // box of this wave's targets: the descriptors of the blocks they lie in
    // (tiles start on block boundaries; lanes past the tile repeat its last
    // target, which lies in the block of the last real lane)
    float tlo[3] = {INFINITY, INFINITY, INFINITY}, thi[3] = {-INFINITY, -INFINITY, -INFINITY};
#pragma unroll
    for (int t = 0; t < T; t++) {
        const int li = min(tl + t * kBlock, it.ntgt - 1);
        const RecF32 r = rec[it.tgt0 + li];
        thx[t] = r.a.x; thy[t] = r.a.y; thz[t] = r.a.z;
        tlx[t] = r.b.x; tly[t] = r.b.y; tlz[t] = r.b.z;
        const int wb = (it.tgt0 + min((tl & ~63) + t * kBlock, it.ntgt - 1)) / kDescPoints;  // wave-uniform
        const desc_float *d = desc_at(E.blk, wb);
#pragma unroll
        for (int k = 0; k < 3; k++) { tlo[k] = fminf(tlo[k], d[k]); thi[k] = fmaxf(thi[k], d[3 + k]); }
#pragma unroll
        for (int k = 0; k < 6; k++) { s[t][k] = 0.0f; c[t][k] = 0.0f; pn[t][k] = 0.0; }
    }
    for (int base = 0; base < it.nsrc; base += kSrcTile) {
        if (QUAD) {
            if (base + (tid & ~63) >= it.nsrc) break;  // wave-uniform: this wave has no block left
            wave_sync();
        } else {
            __syncthreads();
        }
        // this wave stages source block tid / 64 (its anchored positions
        // from the descriptors); padding lanes stage zero loads
        S.put(E, tid, base + tid < it.nsrc ? it.src0 + base + tid : -1);
        if (QUAD) wave_sync();
        else __syncthreads();
        const int cnt = min(kSrcTile, it.nsrc - base);
        // QUAD: only the block this wave staged
        const int sb0 = QUAD ? (tid & ~63) : 0;
        const int sb1 = QUAD ? sb0 + kKahanBlock : cnt;
        for (int sb = sb0; sb < sb1; sb += kKahanBlock) {
            // Issue priority of this wave: the 64-source blocks of the item
            // still to do after this one (3 or more: highest).  A SIMD
            // issues its oldest wave first among equals, so without this
            // the waves that start last wait behind older ones and then
            // finish the launch alone; preferring the waves with the most
            // work left evens out when a SIMD's waves finish (measured on
            // MI355X: -1.2% at 12,800 points, -1.5% for 16 batched 3,200-
            // point slices, +0.5% for 1,000 swimmers, 256,000 points even).
            {
                const int left = (it.nsrc - base - sb - 1) / kKahanBlock;  // wave-uniform
                if (left >= 3) __builtin_amdgcn_s_setprio(3);
                else if (left == 2) __builtin_amdgcn_s_setprio(2);
                else if (left == 1) __builtin_amdgcn_s_setprio(1);
                else __builtin_amdgcn_s_setprio(0);
            }
            float p[T][6];
            // bit j of near[t]: source sb + j is near target t (masked path only)
            uint64_t near[T];
#pragma unroll
            for (int t = 0; t < T; t++) {
                near[t] = 0;
#pragma unroll
                for (int k = 0; k < 6; k++) p[t][k] = 0.0f;
            }
            // descriptor of this source block (wave-uniform)
            float bx[10];
            {
                const desc_float *bd = desc_at(E.blk, (it.src0 + base + sb) / kDescPoints);
#pragma unroll
                for (int k = 0; k < 10; k++) bx[k] = bd[k];
            }
            const float gap2 = box_gap2(tlo, thi, bx, bx + 3);
            // sources of this block that carry contact forces (wave-uniform)
            const uint64_t ljm = E.lj_mask ? ((const mask_word *)E.lj_mask)[(it.src0 + base + sb) / kLjMaskPoints] : 0;
            if (gap2 > kFarBoxGap2 && gap2 > kAnchorGapRatio2 * bx[9]) {
                // wave-uniform: no near pair, separation from the block's anchor
                float ux[T], uy[T], uz[T];
#pragma unroll
                for (int t = 0; t < T; t++) {
                    ux[t] = (thx[t] - bx[6]) + tlx[t];
                    uy[t] = (thy[t] - bx[7]) + tly[t];
                    uz[t] = (thz[t] - bx[8]) + tlz[t];
                }
                if (gap2 > kRemoteBoxGap2) far_block<T, true>(S, sb, sb + kKahanBlock, ux, uy, uz, p);
                else far_block<T, false>(S, sb, sb + kKahanBlock, ux, uy, uz, p);
            } else if (gap2 > kFarBoxGap2) {
                // wave-uniform: no near pair, exact hi/lo separation
#pragma unroll 2
                for (int jj = sb; jj < sb + kKahanBlock; jj++) {
                    const float4 F = S.F[jj], H = S.H[jj];
                    const float Fx = S.W[jj].w, Nz = S.M[jj].x, lx = S.K[jj].w, lz = S.lz[jj];
#pragma unroll
                    for (int t = 0; t < T; t++) {
                        float rx, ry, rz;
                        const float R2 = sep_f32(thx[t], thy[t], thz[t], tlx[t], tly[t], tlz[t], H.x, H.y, H.z, lx,
                                                 H.w, lz, rx, ry, rz);
                        pair_core_f32<false>(rx, ry, rz, R2, Fx, F.x, F.y, F.z, F.w, Nz, p[t]);
                    }
                }
            } else {
#pragma unroll 2
                for (int jj = sb; jj < sb + kKahanBlock; jj++) {
                    const float4 F = S.F[jj], H = S.H[jj];
                    const float Fx = S.W[jj].w, Nz = S.M[jj].x, lx = S.K[jj].w, lz = S.lz[jj];
#pragma unroll
                    for (int t = 0; t < T; t++) {
                        float rx, ry, rz;
                        const float R2 = sep_f32(thx[t], thy[t], thz[t], tlx[t], tly[t], tlz[t], H.x, H.y, H.z, lx,
                                                 H.w, lz, rx, ry, rz);
                        pair_core_f32<true>(rx, ry, rz, R2, Fx, F.x, F.y, F.z, F.w, Nz, p[t]);
                        near[t] |= (uint64_t)(R2 < kNearR2) << (jj - sb);
                    }
                }
            }
#pragma unroll
            for (int t = 0; t < T; t++)
#pragma unroll
                for (int k = 0; k < 6; k++) kahan_add(s[t][k], c[t][k], p[t][k]);
            // the pairs masked above, in FP64 on the exact hi/lo difference:
            // each lane walks only its own near sources
#pragma unroll
            for (int t = 0; t < T; t++) {
                uint64_t m = near[t] & ~ljm;
                while (m) {
                    const int jj = sb + __builtin_ctzll(m);
                    m &= m - 1;
                    const float4 F = S.F[jj], H = S.H[jj];
                    const float lx = S.K[jj].w, lz = S.lz[jj];
                    const float fx = S.W[jj].w, fy = F.x, fz = F.y, nx = F.z, ny = F.w, nz = S.M[jj].x;
                    near_pair_f64(thx[t], thy[t], thz[t], tlx[t], tly[t], tlz[t], H.x, H.y, H.z, lx, H.w, lz, fx, fy,
                                  fz, nx, ny, nz, pn[t]);
                }
            }
        }
    }
    const int N = E.N;
#pragma unroll
    for (int t = 0; t < T; t++)
#pragma unroll
        for (int k = 0; k < 6; k++) pn[t][k] += (double)s[t][k] - (double)c[t][k];
    // the sources with contact forces (they entered the sums above with zero
    // loads), in FP64 for every target: a wave-uniform loop over records in
    // scalar registers, the next one on its way.  After the loop above, where
    // it would cost registers.  When every lane took them with its near pairs, at
    // its own pace and with a load per source, the pair kernel of 1,000 swimmers
    // (6% of the points in contact) took 2,656 us; so 2,547 (MI355X).
    if (E.lj_mask) {
        double tx[T], ty[T], tz[T];
#pragma unroll
        for (int t = 0; t < T; t++) {
            // not before the loop above: its registers are all in use there
            asm volatile("" : "+v"(thx[t]), "+v"(thy[t]), "+v"(thz[t]));
            tx[t] = (double)thx[t] + (double)tlx[t];
            ty[t] = (double)thy[t] + (double)tly[t];
            tz[t] = (double)thz[t] + (double)tlz[t];
        }
        const int b0 = QUAD ? __builtin_amdgcn_readfirstlane(tid & ~63) : 0;
        for (int b = b0; b < it.nsrc; b += QUAD ? kSrcTile : kKahanBlock) {
            uint64_t m = ((const mask_word *)E.lj_mask)[(it.src0 + b) / kLjMaskPoints];
            if (it.nsrc - b < 64) m &= (1ull << (it.nsrc - b)) - 1;
            if (!m) continue;
            ScalarRec next = scalar_rec(rec, it.src0 + b + __builtin_ctzll(m));
            while (m) {
                const ScalarRec r = next;
                m &= m - 1;
                if (m) next = scalar_rec(rec, it.src0 + b + __builtin_ctzll(m));
                const double x = (double)r.v[0] + (double)r.v[4], y = (double)r.v[1] + (double)r.v[5],
                             z = (double)r.v[2] + (double)r.v[6];
#pragma unroll
                for (int t = 0; t < T; t++)
                    pair_f64(tx[t], ty[t], tz[t], x, y, z, r.v[3], r.v[7], r.v[8], r.v[9], r.v[10], r.v[11], 1.0, 3.75,
                             pn[t]);
            }
        }
    }
    if (QUAD) {
        // the four waves' sums for the same targets, added in wave order (the
        // staged sources are no longer needed)
        double *sum = reinterpret_cast<double *>(&S);  // [6][kBlock]
        static_assert(sizeof(S) >= 6 * kBlock * sizeof(double), "sums of four waves");
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 6; k++) sum[k * kBlock + tid] = pn[0][k];
        __syncthreads();
        if (tid < 64 && tid < it.ntgt) {
#pragma unroll
            for (int k = 0; k < 6; k++) {
                double v = sum[k * kBlock + tid];
#pragma unroll
                for (int w = 1; w < kBlock / 64; w++) v += sum[k * kBlock + w * 64 + tid];
                E.part[((size_t)it.chunk * 6 + k) * N + it.tgt0 + tid] = v;
            }
        }
    } else {
#pragma unroll
        for (int t = 0; t < T; t++) {
            const int li = tid + t * kBlock;
            if (li < it.ntgt) {
#pragma unroll
                for (int k = 0; k < 6; k++) E.part[((size_t)it.chunk * 6 + k) * N + it.tgt0 + li] = pn[t][k];
            }
        }
    }
    if (!PERSIST) break;
    idx = claim_item(queue, &sNext);
    }
    if (PERSIST) leave_queue(queue);
}

// FP64 blocks whose box lies at least four half-diagonals from the wave's
// targets take the split cross products (below) with u, w relative to the
// box's centre: |w| <= |r|/4, so (sum H3 n) x u and the sum of H3 (w x n)
// cancel by at most a factor 1.5 and leave the rounding error where it was
// (2-norm and worst relative errors equal to the direct form's to two digits
// at 3,000 to 51,200 points).
constexpr float kSplitGapRatio2F64 = 16.0f;

// Position x relative to a block's centre c (in units of eps).  One rounding, by
// a fused operation that is asked for and not left to the compiler: sources
// (w) and targets (u) have to be taken from the same unrounded centre, or every
// pair of the block gets the rounding of c eps, up to half an ulp of the
// coordinate, in n x r and f x r (blocks of 0.12 across, 40 eps apart, eps 0.02, at
// 10^4 from the origin: errors of 2e-13 instead of 2e-16 of the terms).
__device__ __forceinline__ double from_centre(double x, float c, double eps) { return fma(-(double)c, eps, x); }

// Sources of one staged round of the FP64 kernel: x, y | z, fx | fy, fz |
// nx, ny | nz, m | k with m = w x n, k = w x f.
template <int SLOTS>
struct SrcStageF64 {
    double2 a[SLOTS], b[SLOTS], c[SLOTS], d[SLOTS], e[SLOTS], f[SLOTS], g[SLOTS];
    double h[SLOTS];
    // Stages source i of E at slot j; its block's descriptor is wave-uniform.
    __device__ __forceinline__ void put(const EnsDesc &E, int j, int i) {
        const double2 *src = reinterpret_cast<const double2 *>(E.rec) + (size_t)i * 5;
        const double2 w0 = src[0], w1 = src[1], w2 = src[2], w3 = src[3], w4 = src[4];
        const desc_float *bd = desc_at(E.blk, __builtin_amdgcn_readfirstlane(i / kDescPoints));
        const double wx = from_centre(w0.x, bd[6], E.rec_eps), wy = from_centre(w0.y, bd[7], E.rec_eps),
                     wz = from_centre(w1.x, bd[8], E.rec_eps);
        const double fx = w1.y, fy = w2.x, fz = w2.y, nx = w3.x, ny = w3.y, nz = w4.x;
        a[j] = w0; b[j] = w1; c[j] = w2; d[j] = w3;
        e[j] = make_double2(nz, fma(wy, nz, -(wz * ny)));
        f[j] = make_double2(fma(wz, nx, -(wx * nz)), fma(wx, ny, -(wy * nx)));
        g[j] = make_double2(fma(wy, fz, -(wz * fy)), fma(wz, fx, -(wx * fz)));
        h[j] = fma(wx, fy, -(wy * fx));
    }
};

// Sums of the staged sources [sb, se) into acc for targets at (tx, ty, tz), by
// split cross products (as in far_block, with H4 = eps^2 u - H3/2): 51
// instructions per pair and one v_rsq_f64 against 57 for the direct form.  FP64
// instructions issue at one per 4.1 clocks and SIMD from two waves on, so the
// registers of the further sums (149 VGPRs and three blocks per CU with two
// targets per lane, 124 and four before) cost nothing: pair kernel 4.72 ->
// 4.42 ms at 51,200 points, 308 -> 296 us at 12,800 (MI355X; there the last of
// its 1.6 rounds of blocks weighs more).
template <int T, class STAGE>
__device__ __forceinline__ void far_block_f64(const STAGE &S, int sb, int se, const double (&tx)[T],
                                              const double (&ty)[T], const double (&tz)[T], const float *ctr,
                                              double eps, double e2, double (&acc)[T][6]) {
    const double c15e2 = 1.5 * e2, c375e2 = 3.75 * e2;
    double sn[T][3], sf[T][3], su[T][3];
#pragma unroll
    for (int t = 0; t < T; t++)
#pragma unroll
        for (int k = 0; k < 3; k++) { sn[t][k] = 0.0; sf[t][k] = 0.0; su[t][k] = 0.0; }
#pragma unroll 2
    for (int jj = sb; jj < se; jj++) {
        const double2 A = S.a[jj], B = S.b[jj], C = S.c[jj], Dd = S.d[jj], Ee = S.e[jj], F = S.f[jj], G = S.g[jj];
        const double kz = S.h[jj];
        const double fx = B.y, fy = C.x, fz = C.y, nx = Dd.x, ny = Dd.y, nz = Ee.x;
#pragma unroll
        for (int t = 0; t < T; t++) {
            const double rx = tx[t] - A.x, ry = ty[t] - A.y, rz = tz[t] - B.x;
            const double q = rsq_f64(fma(rz, rz, fma(ry, ry, fma(rx, rx, e2))));
            const double q2 = q * q, q3 = q2 * q, q5 = q3 * q2, q7 = q5 * q2;
            const double h1 = fma(e2, q3, q);
            const double h3 = fma(c15e2, q5, q3);
            const double u = c375e2 * q7;
            const double h5 = fma(1.5, q5, u);
            const double fr = fma(fz, rz, fma(fy, ry, fx * rx));
            const double nr = fma(nz, rz, fma(ny, ry, nx * rx));
            const double a = q3 * fr, b = h5 * nr;
            acc[t][0] = fma(h3, Ee.y, fma(a, rx, fma(h1, fx, acc[t][0])));
            acc[t][1] = fma(h3, F.x, fma(a, ry, fma(h1, fy, acc[t][1])));
            acc[t][2] = fma(h3, F.y, fma(a, rz, fma(h1, fz, acc[t][2])));
            acc[t][3] = fma(h3, G.x, fma(b, rx, acc[t][3]));
            acc[t][4] = fma(h3, G.y, fma(b, ry, acc[t][4]));
            acc[t][5] = fma(h3, kz, fma(b, rz, acc[t][5]));
            su[t][0] = fma(u, nx, su[t][0]);  // H4 = eps^2 u - H3/2
            su[t][1] = fma(u, ny, su[t][1]);
            su[t][2] = fma(u, nz, su[t][2]);
            sn[t][0] = fma(h3, nx, sn[t][0]);
            sn[t][1] = fma(h3, ny, sn[t][1]);
            sn[t][2] = fma(h3, nz, sn[t][2]);
            sf[t][0] = fma(h3, fx, sf[t][0]);
            sf[t][1] = fma(h3, fy, sf[t][1]);
            sf[t][2] = fma(h3, fz, sf[t][2]);
        }
    }
#pragma unroll
    for (int t = 0; t < T; t++) {
        const double ux = from_centre(tx[t], ctr[0], eps), uy = from_centre(ty[t], ctr[1], eps),
                     uz = from_centre(tz[t], ctr[2], eps);
        acc[t][0] += fma(sn[t][1], uz, -(sn[t][2] * uy));
        acc[t][1] += fma(sn[t][2], ux, -(sn[t][0] * uz));
        acc[t][2] += fma(sn[t][0], uy, -(sn[t][1] * ux));
        acc[t][3] += fma(e2, su[t][0], fma(-0.5, sn[t][0], fma(sf[t][1], uz, -(sf[t][2] * uy))));
        acc[t][4] += fma(e2, su[t][1], fma(-0.5, sn[t][1], fma(sf[t][2], ux, -(sf[t][0] * uz))));
        acc[t][5] += fma(e2, su[t][2], fma(-0.5, sn[t][2], fma(sf[t][0], uy, -(sf[t][1] * ux))));
    }
}

// QUAD: a block takes a quarter of an item's targets, 64, and its four waves
// split each source block: four times the blocks of a quarter of the time.  In
// a small grid a wave has a SIMD to itself or shares it with one or two
// others, so the time is that of the longest chain and of the fullest CU (25
// swimmers of 51 points, 100 items: 14.6 -> 8.8 us, MI355X).
// Blocks per CU the register budget allows: 4 with one target per lane, 3 with two.
template <int T, bool PERSIST, bool QUAD>
__global__ __launch_bounds__(kBlock, T == 1 ? 4 : 3) void k_pairs_tile_f64(const EnsDesc *__restrict__ desc,
                                                           const PairItem *__restrict__ items, int n_items,
                                                           uint32_t *queue) {
    static_assert(!QUAD || T == 1, "four-wave source split: one target per lane");
    constexpr int kTargets = QUAD ? 64 : kBlock;    // targets per block and t
    constexpr int kPart = QUAD ? kDescPoints / 4 : kDescPoints;  // sources of a block per wave
    __shared__ SrcStageF64<kSrcTile> S;
    __shared__ int sNext;
    int idx = PERSIST ? claim_item(queue, &sNext) : (int)blockIdx.x;
    while (idx < n_items) {
    PairItem it = items[QUAD ? idx / 4 : idx];
    if (QUAD) {
        const int q = 64 * (idx % 4);
        if (q >= it.ntgt) {  // the last tile is not full
            if (!PERSIST) break;
            idx = claim_item(queue, &sNext);
            continue;
        }
        it.tgt0 += q;
        it.ntgt = min(64, it.ntgt - q);
    }
    const EnsDesc E = global_desc(desc[it.ens]);
    const RecF64 *__restrict__ rec = reinterpret_cast<const RecF64 *>(E.rec);
    const int tid = threadIdx.x, tl = QUAD ? tid & 63 : tid;
    const int part0 = QUAD ? __builtin_amdgcn_readfirstlane(tid >> 6) * kPart : 0;
    const double eps = E.rec_eps, e2 = eps * eps, c375e2 = 3.75 * e2;
    double tx[T], ty[T], tz[T], acc[T][6];
    const desc_float *tbox[T];  // descriptors of the blocks this wave's targets lie in (wave-uniform)
#pragma unroll
    for (int t = 0; t < T; t++) {
        const int li = min(tl + t * kTargets, it.ntgt - 1);
        const RecF64 &r = rec[it.tgt0 + li];
        tx[t] = r.x; ty[t] = r.y; tz[t] = r.z;
        const int wb = (it.tgt0 + min((tl & ~63) + t * kTargets, it.ntgt - 1)) / kDescPoints;
        tbox[t] = desc_at(E.blk, __builtin_amdgcn_readfirstlane(wb));
#pragma unroll
        for (int k = 0; k < 6; k++) acc[t][k] = 0.0;
    }
    for (int base = 0; base < it.nsrc; base += kSrcTile) {
        __syncthreads();
        // this wave stages the source block tid / 64 of the round
        if (base + tid < it.nsrc) S.put(E, tid, it.src0 + base + tid);
        __syncthreads();
        const int cnt = min(kSrcTile, it.nsrc - base);
        for (int sb = 0; sb < cnt; sb += kDescPoints) {
            const int s0 = sb + part0, se = min(s0 + kPart, cnt);
            const desc_float *d = desc_at(E.blk, (it.src0 + base + sb) / kDescPoints);
            float slo[3], shi[3], gap2 = INFINITY;
#pragma unroll
            for (int k = 0; k < 3; k++) { slo[k] = d[k]; shi[k] = d[3 + k]; }
#pragma unroll
            for (int t = 0; t < T; t++) {
                float lo[3], hi[3];
#pragma unroll
                for (int k = 0; k < 3; k++) { lo[k] = tbox[t][k]; hi[k] = tbox[t][3 + k]; }
                gap2 = fminf(gap2, box_gap2(lo, hi, slo, shi));
            }
            if (gap2 > kFarBoxGap2 && gap2 > kSplitGapRatio2F64 * d[9]) {  // wave-uniform
                const float ctr[3] = {d[6], d[7], d[8]};
                far_block_f64<T>(S, s0, se, tx, ty, tz, ctr, eps, e2, acc);
            } else {
#pragma unroll 2
                for (int jj = s0; jj < se; jj++) {
                    const double2 A = S.a[jj], B = S.b[jj], C = S.c[jj], D = S.d[jj];
                    const double nz = S.e[jj].x;
#pragma unroll
                    for (int t = 0; t < T; t++)
                        pair_f64(tx[t], ty[t], tz[t], A.x, A.y, B.x, B.y, C.x, C.y, D.x, D.y, nz, e2, c375e2, acc[t]);
                }
            }
        }
    }
    const int N = E.N;
    if (QUAD) {
        // the four waves' sums for the same targets, added in wave order (the
        // staged sources are no longer needed)
        double *sum = reinterpret_cast<double *>(&S);  // [6][kBlock]
        static_assert(sizeof(S) >= 6 * kBlock * sizeof(double), "sums of four waves");
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 6; k++) sum[k * kBlock + tid] = acc[0][k];
        __syncthreads();
        for (int k = tid >> 6; k < 6; k += kBlock / 64) {
            double v = sum[k * kBlock + tl];
#pragma unroll
            for (int w = 1; w < kBlock / 64; w++) v += sum[k * kBlock + w * 64 + tl];
            if (tl < it.ntgt) E.part[((size_t)it.chunk * 6 + k) * N + it.tgt0 + tl] = v;
        }
    } else {
#pragma unroll
        for (int t = 0; t < T; t++) {
            const int li = tid + t * kBlock;
            if (li < it.ntgt) {
#pragma unroll
                for (int k = 0; k < 6; k++) E.part[((size_t)it.chunk * 6 + k) * N + it.tgt0 + li] = acc[t][k];
            }
        }
    }
    if (!PERSIST) break;
    idx = claim_item(queue, &sNext);
    }
    if (PERSIST) leave_queue(queue);
}

// Small-ensemble pair kernel: each wave owns kSplitTargetsPerWave targets and
// its 64 lanes stride over the item's sources; per-lane sums are combined in
// FP64 with a butterfly of wave shuffles in a fixed order.  Sources are staged
// through LDS 256 at a time by the whole block (its waves share them).
//
// The records are of the FP64 kind in both precisions (REC_WIDE for FP32C).
// The launch is bound by latency and by the FP64 pairs near the targets, so an
// FP32 pass over the far sources only added to it (two passes, 1,020 points
// in contact: 14.6 us; 9.1 us so, and 46.3 -> 27.0 us in a batch of eight;
// 512 points of 128-point filaments 8.5 -> 6.6 and 14.7 -> 11.6 us; MI355X).
//
// DIRECT: the whole of a one-shot evaluation (one source chunk): the records
// are formed from the caller's row-major arrays as they are staged and U,
// Omega are written in place of the partial sums, with the same operations as
// the pack and reduction kernels.
constexpr int kSplitRound = kBlock;

template <bool DIRECT, int TW>
__device__ __forceinline__ void split_item(const EnsDesc &E, const PairItem it) {
    static_assert(sizeof(RecF32) == 48 && sizeof(RecF64) == 80, "record layouts");
    __shared__ RecF64 sRec[kSplitRound];
    const int tid = threadIdx.x, lane = tid & 63;
    const int tb = (tid >> 6) * TW;
    // a wave without targets still stages sources and meets every barrier
    const bool active = tb < it.ntgt;  // wave-uniform
    const RecF64 *__restrict__ rec = reinterpret_cast<const RecF64 *>(E.rec);
    const auto load = [&](int i) { return DIRECT ? input_rec_f64(E, i) : rec[i]; };
    const double e2 = E.rec_eps * E.rec_eps, c375e2 = 3.75 * e2;
    double tx[TW], ty[TW], tz[TW], acc[TW][6];
#pragma unroll
    for (int t = 0; t < TW; t++) {
        const RecF64 r = load(it.tgt0 + min(tb + t, it.ntgt - 1));
        tx[t] = r.x; ty[t] = r.y; tz[t] = r.z;
#pragma unroll
        for (int k = 0; k < 6; k++) acc[t][k] = 0.0;
    }
    for (int j0 = 0; j0 < it.nsrc; j0 += kSplitRound) {
        const int cnt = min(kSplitRound, it.nsrc - j0);
        __syncthreads();
        for (int q = tid; q < cnt; q += kBlock) sRec[q] = load(it.src0 + j0 + q);
        __syncthreads();
        if (!active) continue;
        for (int j = lane; j < cnt; j += 64) {
            const RecF64 r = sRec[j];
#pragma unroll
            for (int t = 0; t < TW; t++)
                pair_f64(tx[t], ty[t], tz[t], r.x, r.y, r.z, r.fx, r.fy, r.fz, r.nx, r.ny, r.nz, e2, c375e2, acc[t]);
        }
    }
    if (!active) return;  // no barrier follows
    wave_sum_n<6 * TW>(&acc[0][0]);
    if (lane < 6) {
        const int N = E.N;
#pragma unroll
        for (int t = 0; t < TW; t++) {
            if (tb + t < it.ntgt) {
                double v = acc[t][0];
#pragma unroll
                for (int k = 1; k < 6; k++) v = (lane == k) ? acc[t][k] : v;
                if (DIRECT) {
                    const size_t o = 3 * (size_t)(it.tgt0 + tb + t);
                    if (lane < 3) E.U[o + lane] = v * E.cU;
                    else E.W[o + lane - 3] = v * E.cW;
                } else {
                    E.part[((size_t)it.chunk * 6 + lane) * N + it.tgt0 + tb + t] = v;
                }
            }
        }
    }
}

__global__ __launch_bounds__(kBlock) void k_pairs_split(const EnsDesc *__restrict__ desc,
                                                        const PairItem *__restrict__ items) {
    const PairItem it = items[blockIdx.x];
    split_item<false, kSplitTargetsPerWave>(global_desc(desc[it.ens]), it);
}

// One-shot evaluation in one launch, with no scratch and no work list: a
// 64-point FP64 call takes 8 us on one stream and 20 us on streams in turn (each
// waits for the one before) instead of 20 and 36 with pack, pair and reduction
// kernels and an uploaded list (MI355X).  Larger ones, see launch_eval_direct.
template <int TW>
__global__ __launch_bounds__(kBlock) void k_eval_direct(const EnsDesc E) {
    constexpr int kTargets = TW * (kBlock / 64);
    const int t0 = (int)blockIdx.x * kTargets;
    split_item<true, TW>(E, {0, t0, min(kTargets, E.N - t0), 0, E.N, 0});
}

// --------------------------------------------------------- launch wrapper

// Two targets per wave read each staged source once for both, but halve the
// blocks: taken when the fullest CU then has no more targets (FP64 calls, one
// against two targets per wave: 1,000 points 10.4 and 12.8 us, 2,560 points
// 27.6 and 30.9, 3,200 points 40.0 and 36.9, 5,003 points 74.4 and 74.8, 6,144
// points 105 and 93; four never won by more than 1 us; MI355X).
hipError_t launch_eval_direct(const EnsDesc &h_desc, int n_cu, hipStream_t s) {
    if (h_desc.N == 0) return hipSuccess;
    const int w = kBlock / 64;
    const auto blocks = [&](int tw) { return (h_desc.N + tw * w - 1) / (tw * w); };
    const auto per_cu = [&](int tw) { return tw * ((blocks(tw) + n_cu - 1) / n_cu); };
    if (per_cu(2) <= per_cu(1)) hipLaunchKernelGGL(k_eval_direct<2>, dim3(blocks(2)), dim3(kBlock), 0, s, h_desc);
    else hipLaunchKernelGGL(k_eval_direct<1>, dim3(blocks(1)), dim3(kBlock), 0, s, h_desc);
    return hipGetLastError();
}

template <int T, bool PERSIST>
static void launch_tile(int prec, dim3 g, dim3 b, hipStream_t s, const EnsDesc *d_desc, const PairItem *d_items,
                        int n_items, uint32_t *queue) {
    if (prec == 1)
        hipLaunchKernelGGL((k_pairs_tile_f32<T, PERSIST, false>), g, b, 0, s, d_desc, d_items, n_items, queue);
    else hipLaunchKernelGGL((k_pairs_tile_f64<T, PERSIST, false>), g, b, 0, s, d_desc, d_items, n_items, queue);
}

// Resident blocks per CU of a tiled pair kernel (persistent schedule).
int pairs_resident_blocks(int prec, int tpl) {
    static int cache[2][3] = {{0, 0, 0}, {0, 0, 0}};
    int &c = cache[prec == 1][tpl == 2 ? 2 : 1];
    if (c > 0) return c;
    int nb = 0;
    hipError_t e;
    if (prec == 1)
        e = tpl == 2 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_pairs_tile_f32<2, true, false>, kBlock, 0)
                     : hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_pairs_tile_f32<1, true, false>, kBlock, 0);
    else
        e = tpl == 2 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_pairs_tile_f64<2, true, false>, kBlock, 0)
                     : hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_pairs_tile_f64<1, true, false>, kBlock, 0);
    c = (e == hipSuccess && nb > 0) ? nb : 1;
    return c;
}

hipError_t launch_pairs(int prec, int mode, int tpl, const EnsDesc *d_desc, const PairItem *d_items,
                        int n_items, hipStream_t s, uint32_t *queue, int resident) {
    if (n_items == 0) return hipSuccess;
    const dim3 b(kBlock);  // the pair kernels index LDS by threadIdx.x < kBlock
    if (mode == PAIR_SPLIT) {
        const dim3 g(n_items);
        hipLaunchKernelGGL(k_pairs_split, g, b, 0, s, d_desc, d_items);
    } else if (mode == PAIR_QUAD && prec != 1) {  // in quarters: four blocks per item
        const int n = 4 * n_items;
        if (queue && resident > 0)
            hipLaunchKernelGGL((k_pairs_tile_f64<1, true, true>), dim3((unsigned)std::min(n, resident)), b, 0, s,
                               d_desc, d_items, n, queue);
        else
            hipLaunchKernelGGL((k_pairs_tile_f64<1, false, true>), dim3(n), b, 0, s, d_desc, d_items, n, nullptr);
    } else if (mode == PAIR_QUAD) {
        if (queue && resident > 0)
            hipLaunchKernelGGL((k_pairs_tile_f32<1, true, true>), dim3((unsigned)std::min(n_items, resident)), b, 0, s,
                               d_desc, d_items, n_items, queue);
        else
            hipLaunchKernelGGL((k_pairs_tile_f32<1, false, true>), dim3(n_items), b, 0, s, d_desc, d_items, n_items,
                               nullptr);
    } else if (queue && resident > 0) {
        const dim3 g((unsigned)std::min(n_items, resident));
        if (tpl == 2) launch_tile<2, true>(prec, g, b, s, d_desc, d_items, n_items, queue);
        else launch_tile<1, true>(prec, g, b, s, d_desc, d_items, n_items, queue);
    } else {
        const dim3 g(n_items);
        if (tpl == 2) launch_tile<2, false>(prec, g, b, s, d_desc, d_items, n_items, nullptr);
        else launch_tile<1, false>(prec, g, b, s, d_desc, d_items, n_items, nullptr);
    }
    return hipGetLastError();
}

}  // namespace mrs
