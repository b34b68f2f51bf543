// Internal types shared by the HIP kernels and the host runtime.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mrs {

// Threads per block of every kernel on the path (4 wave64s).
constexpr int kBlock = 256;
// Sources staged in LDS per tile of the tiled pair kernel.
constexpr int kSrcTile = 256;
// Sources summed in plain FP32 before one compensated (Kahan) update.
constexpr int kKahanBlock = 64;
// Targets per wave in the small-N pair kernel (lanes split the sources).
// One: the kernel is latency-bound, and four times the waves shorten each
// wave's chain (MI355X, FP64 records, which both precisions use: 64 points 8.2 ->
// 6.3 us, 960 points 19.1 -> 11.8; same results, since each target's sum is formed
// the same way).
constexpr int kSplitTargetsPerWave = 1;
constexpr int kSplitTargetsPerBlock = kSplitTargetsPerWave * (kBlock / 64);

// Source record of the FP32C pair kernel, 48 bytes, read as three float4:
//   a = (xh, yh, zh, fx)  b = (xl, yl, zl, fy)  c = (fz, nx, ny, nz)
// with positions scaled by 1/eps and split hi + lo, forces scaled by 1/eps
// and torques by 1/eps^2.
struct alignas(16) RecF32 {
    float4 a, b, c;
};

// Source record of the FP64 pair kernel, 80 bytes (five 16-byte words).
struct alignas(16) RecF64 {
    double x, y, z, fx, fy, fz, nx, ny, nz, pad;
};

// Form of an ensemble's source records.  REC_WIDE holds the values of the
// FP32C records (hi + lo, which is exact in double, and the FP32 loads) in
// FP64 records, for FP32C ensembles that the FP64 kernels sum faster; units of
// eps, like REC_F32.
enum RecForm : int { REC_F64 = 0, REC_F32 = 1, REC_WIDE = 2 };

// Source-block descriptor of the tiled pair kernels (one per aligned 64-point
// block, in units of eps), padded to 64 bytes.
constexpr int kDescFloats = 16;
constexpr int kDescPoints = 64;

// Bytes of a record buffer for n points in either precision: FP64 records, or
// FP32C records followed by the anchored positions; then the block
// descriptors.
inline size_t rec_buffer_bytes(int64_t n) {
    static_assert(sizeof(RecF64) >= sizeof(RecF32) + sizeof(float4), "the FP64 form is the larger one");
    return (size_t)n * sizeof(RecF64) +
           (size_t)((n + kDescPoints - 1) / kDescPoints) * kDescFloats * sizeof(float);
}

// Everything a kernel needs to know about one ensemble.  Arrays are SoA:
// component c of point i of an N-point vector field lives at [c * N + i];
// director i, component c of point k at [(3 i + c) * N + k].
struct EnsDesc {
    int32_t N;
    int32_t n_fil;
    int32_t K;         // source chunks of the split-K pair kernel
    int32_t aos_io;    // 1: X/f/n inputs and U/W outputs are n x 3 row-major
    const int32_t *off;
    double *X, *D;     // state (SoA)
    double *Xs, *Ds;   // RK stage state (SoA)
    double *U, *W;     // velocities (SoA, or AoS when aos_io)
    double *Ua, *Wa;   // RK weighted sums (SoA)
    double *Ks;        // RK4: the last stage's corrected angular velocity k (SoA)
    const double *fext, *next;  // external loads (SoA, or AoS when aos_io), may be null
    const double *Xin_aos;      // AoS positions when aos_io
    void *rec;         // source records (RecF32 or RecF64), N entries
    int32_t form;      // RecForm of the records
    // tiled pair kernels: per aligned 64-point block the descriptor
    // (kDescFloats floats, in units of eps: widened hi-part box lo[3], hi[3],
    // centre[3], squared half-diagonal), and for FP32C per point its position
    // relative to the centre of its block (anchored form); both follow the
    // records in the same buffer (set_records) and are written with them
    // (k_rod_forces descriptor items, k_pack_aos)
    float4 *wanch;
    float *blk;
    double *part;      // split-K partial sums [K][6][N]
    double *g_out, *m_out;  // rod loads, row-major (k_rod_forces_aos)
    double eps, inv_eps, mu;
    double rec_eps;    // eps in the units of FP64-kind records: eps (REC_F64) or 1 (REC_WIDE)
    double cU, cW;     // 1/(8 pi mu) and the Omega scale of the record form
    double a[3], b[3], om0[3], ds;
    double dt;         // step size used when a launch passes dt = NaN
    int32_t elastic;   // rod forces on/off used when a launch passes elastic < 0
    // swimming (Sec. IV): waveform (A, k, f) added to the preferred
    // strain-twist, Lennard-Jones repulsion between filaments
    int32_t has_wave, has_lj;
    int32_t n_ljblk;        // source blocks of the LJ pass (with LJ)
    double wave[3];
    double lj_sig, lj_e, lj_rc;
    double *clock;          // time at the start of the current step (one double)
    const int32_t *fil;     // filament of each point (with LJ)
    double *flj;            // LJ force on each point [3][N] (with LJ)
    const int32_t *lj_blk;  // per LJ source block: first point, end, filament (with LJ)
    double *lj_box;         // per LJ source block: lo[3], hi[3] of its positions (with LJ)
    uint64_t *lj_mask;      // per aligned 64-point block: bit j set when point 64 b + j
                            // feels a LJ force (with LJ)
    int32_t *nonfinite;     // set to 1 (plain vector store) by the reduction when a
                            // result it writes is not finite; may be null
};

// Source blocks of the Lennard-Jones pass hold at most this many consecutive
// points of one filament; the LJ mask covers aligned blocks of 64 points.
constexpr int kLjBlockPoints = 64;
constexpr int kLjMaskPoints = 64;

// One block of a pair kernel: targets [tgt0, tgt0 + ntgt) against sources
// [src0, src0 + nsrc) of ensemble `ens`, written to split-K chunk `chunk`.
struct PairItem {
    int32_t ens, tgt0, ntgt, src0, nsrc, chunk;
};

// One block of the rod-force kernel: filament `fil` of ensemble `ens`; or,
// with fil = -1 - g (tiled configurations), the source-block
// descriptors of blocks kBlock / 64 * g ... of ensemble `ens`, one per wave.
struct RodItem {
    int32_t ens, fil;
};

// Largest ensembles of k_lj_rods: points (their positions lie in LDS, 24 B
// each) and LJ source blocks (one per lane).
constexpr int kLjRodPoints = 3200, kLjRodBlocks = 64;

// Filament offsets of k_rod_forces_aos: filaments of `step` points each, or
// (step = 0) the offsets themselves, up to kRodArgOffsets of them in the
// kernel's arguments (argument blocks end at 4 KiB), more in a device list.
constexpr int kRodArgOffsets = 800;
struct RodOffsets {
    const int32_t *list;  // device, or null
    int32_t step;
    int32_t v[kRodArgOffsets];
};
static_assert(sizeof(EnsDesc) + sizeof(RodOffsets) <= 4096, "kernel arguments of k_rod_forces_aos");

// Points per block of the reduction/epilogue kernel, and its threads: the
// block's waves split the source chunks of its points.
constexpr int kReducePoints = 64;
constexpr int kReduceThreads = 256;

// One block of the reduction/epilogue kernel: points [p0, p0 + kReducePoints).
struct PointItem {
    int32_t ens, p0;
};

enum Epilogue : int {
    EPI_WRITE = 0,     // U, W only
    EPI_EULER = 1,     // U, W and a forward Euler step
    EPI_RK_STAGE = 2,  // accumulate stage s, build stage state s + 1
    EPI_RK_FINAL = 3,  // accumulate last stage, finish the step
};

// Runge-Kutta schemes of the stage epilogue.
enum RkScheme : int { RK_SCHEME_RK4 = 0, RK_SCHEME_RK2 = 1 };

// Points the records of an ensemble of n points at rec (a buffer of
// rec_buffer_bytes(n)) in the given form; with desc the block descriptors and
// (REC_F32) the anchored positions follow them, otherwise both are null (no
// tiled kernel reads them).
inline void set_records(EnsDesc &d, void *rec, int64_t n, RecForm form, bool desc) {
    d.rec = rec;
    d.form = form;
    d.rec_eps = form == REC_F64 ? d.eps : 1.0;
    char *b = static_cast<char *>(rec);
    const bool f32 = form == REC_F32;
    const size_t r = (size_t)n * (f32 ? sizeof(RecF32) : sizeof(RecF64));
    const size_t w = f32 ? (size_t)n * sizeof(float4) : 0;
    d.wanch = desc && f32 ? reinterpret_cast<float4 *>(b + r) : nullptr;
    d.blk = desc ? reinterpret_cast<float *>(b + r + w) : nullptr;
}

// A part of an evaluation's work list as a kernel argument (k_store_list).
constexpr int kListWords = 240;  // argument blocks end at 4 KiB
struct ListPart {
    uint4 v[kListWords];
};

// Launch wrappers (mrs_pairs.hip, mrs_kernels.hip).  All return the launch's hipError_t.
hipError_t launch_pack_aos(const EnsDesc &h_desc, const void *src, void *dst, size_t bytes, hipStream_t s);
// bytes (a multiple of 16) of host memory to dst by value: once queued, or
// captured, the source is not read again.
hipError_t launch_store_list(const void *src, void *dst, size_t bytes, hipStream_t s);
// elastic < 0: every ensemble uses its own EnsDesc::elastic.  The waveform
// time of the launch is clock + c dt, c the node of RK stage `stage` of
// `scheme` (0 for stage 0); dt = NaN: every ensemble uses its own dt.
hipError_t launch_rod_forces(int stage_state, int elastic, int scheme, int stage, double dt,
                             const EnsDesc *d_desc, const RodItem *d_items, int n_items, hipStream_t s);
// Rod forces of h_desc.n_fil >= 1 filaments on row-major arrays (h_desc.X, D,
// fext, next; g_out, m_out).
hipError_t launch_rod_forces_aos(const EnsDesc &h_desc, const RodOffsets &off, hipStream_t s);
// Lennard-Jones forces of the ensembles with has_lj: the box of every LJ
// source block (box items: (ensemble, first of kBlock / 64 blocks)), then the
// force on every point and the LJ masks (target items: (ensemble, first of
// kLjMaskPoints consecutive points)).
// max_points <= kLjRodPoints: largest ensemble of the items.
hipError_t launch_lj_rods(int stage_state, int elastic, int scheme, int stage, double dt, const EnsDesc *d_desc,
                          const RodItem *d_items, int n_items, int max_points, hipStream_t s);
hipError_t launch_lj(int stage_state, const EnsDesc *d_desc, const PointItem *d_box_items, int n_box_items,
                     const PointItem *d_items, int n_items, hipStream_t s);
// queue (two uint32 that are zero before the launch and zero again after
// it) and resident > 0: tiled kernels run the persistent schedule with
// min(n_items, resident) blocks; otherwise one block per item.
hipError_t launch_pairs(int prec, int mode, int tpl, const EnsDesc *d_desc, const PairItem *d_items,
                        int n_items, hipStream_t s, uint32_t *queue = nullptr, int resident = 0);
// One-shot evaluation in one launch: h_desc's row-major inputs (Xin_aos, fext,
// next) and outputs (U, W), its scales and size; outputs must not overlap
// inputs.  Every block forms all records again, for little (at 2,048 points a
// fortieth of its pair work).
hipError_t launch_eval_direct(const EnsDesc &h_desc, int n_cu, hipStream_t s);
// Resident blocks per CU of the persistent tiled pair kernel.
int pairs_resident_blocks(int prec, int tpl);
// dt = NaN: every ensemble uses its own EnsDesc::dt.
hipError_t launch_reduce(int epi, int stage, int scheme, double dt, const EnsDesc *d_desc,
                         const PointItem *d_items, int n_items, hipStream_t s);
// nsteps steps (kSmallEval: the velocities) of n_ens ensembles of at most
// kSmallPoints points, one workgroup each; scheme: as for launch_rod_forces,
// or one of the two below.
constexpr int kSmallPoints = 64, kSmallThreads = 512, kSmallEuler = -1, kSmallEval = -2;
hipError_t launch_small_steps(int scheme, int nsteps, int elastic, double dt, const EnsDesc *d_desc, int n_ens,
                              hipStream_t s);
hipError_t launch_rotsqrt(int64_t count, const double *R, double *S, hipStream_t s);
// out[0] = shader-clock ticks, out[1] = reference-clock ticks of a spin of `cycles` ticks.
hipError_t launch_clock_probe(int64_t cycles, uint64_t *out, hipStream_t s);
// Parareal correction (SoA states of N points): X = Xf + Xg - Xo, D = reorth(Df + Dg - Do).
hipError_t launch_parareal_correct(int N, const double *Xf, const double *Df, const double *Xg, const double *Dg,
                                  const double *Xo, const double *Do, double *X, double *D, hipStream_t s);

// Row-major host arrays to and from stored SoA arrays: rows [0, n_rows) of the
// chunk are the caller's points i0.., stored at inv[i0 + row].
struct RowArray {
    double *soa;   // device, component c of stored point k at [c N + k]
    double *rows;  // pinned host memory mapped on the device, row-major; null (in): zeros
    int32_t w;     // components, 3 or 9
};
struct RowArrays {
    RowArray a[4];
    int32_t count;
};
hipError_t launch_rows_in(const RowArrays &ra, const int32_t *inv, int64_t N, int64_t i0, int64_t n_rows,
                          hipStream_t s);
// Sets *nonfinite to 1 (plain vector store) when a value copied out is not finite.
hipError_t launch_rows_out(const RowArrays &ra, const int32_t *inv, int64_t N, int64_t i0, int64_t n_rows,
                           int32_t *nonfinite, hipStream_t s);
hipError_t launch_set_value(double *p, double v, hipStream_t s);

// Pair-kernel modes.
// PAIR_QUAD: tiles of 64 targets whose four waves split the sources (FP32C
// items of 64 targets; FP64 in quarters of PAIR_TILE items).
enum PairMode : int { PAIR_TILE = 0, PAIR_SPLIT = 1, PAIR_QUAD = 2 };
// Schedules of the tiled pair kernels: one block per item, or a resident
// grid whose blocks claim items from a queue.
enum PairSched : int { SCHED_GRID = 0, SCHED_PERSISTENT = 1 };
// Work-queue counters per plan: one pair of uint32 per pair-kernel launch
// of a stage (split, tile1, tile2), padded.
constexpr int kQueueWords = 16;

}  // namespace mrs
