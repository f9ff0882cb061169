// Internal declarations shared by the host library and the HIP kernels.
// Not part of the public ABI (see include/tpcf.h).
#pragma once

#include <math.h>
#include <stddef.h>
#include <hip/hip_vector_types.h>
#include <stdint.h>

#include "units.h"

namespace tpcf {

// LDS budget of the cell table; entries are one byte when every slot and
// edge index fits in 7 bits, else two bytes.
constexpr int kMaxLutBytes = 24576;
constexpr int kMaxLutCells = kMaxLutBytes;        // with one-byte entries
// Largest cell-table budget a tuning may ask for.
constexpr int kMaxDirectLutBytes = 33792;
// By default FP32 launches size their cell table so that a block's LDS stays
// within the target: four blocks of four wavefronts in a CU's 160 KiB, the
// occupancy the kernel is compiled for (waves_per_eu_of).
constexpr int kLdsTarget = 40960;
// Wavefronts per SIMD a pair kernel is compiled for: 4 for the FP32 tiles
// (2, 3; two accumulators, eight row operands and the accumulator input in
// at most 128 VGPRs), 5 for the FP64 paths (1, 4).
constexpr int waves_per_eu_of(int path) { return path == 2 || path == 3 ? 4 : 5; }
// FP32 tiles: error bound of q^ in units of 2^-24 (derived in
// docs/fp32_band.md, section 4b): kTileErrN |b|^2 + kTileErrA rho^2 + kTileErr0.
constexpr float kTileErrN = 24.0f;
constexpr float kTileErrA = 640.0f;
constexpr float kTileErr0 = 16.0f;
// Largest e, relative to q^, for which pairs are binned one by one from q^
// (the tiles' cells hold for every q within this of theirs).
constexpr float kTileFar = 1.0f / 1024.0f;
// Work statistics words of a launch (see PairArgs::stats).
constexpr int kStats = 9;
// Their copies in device memory, spread over lines of 128 bytes and summed
// when read.
constexpr int kStatCopies = 32, kStatStride = 16;
constexpr int kStatWords = kStatCopies * kStatStride;
// Counters the work items of a launch are dealt to, on lines of 128 bytes.
constexpr uint32_t kQueues = 8, kQueueStride = 32;
constexpr int kQueueWords = kQueues * kQueueStride / 2;     // u64
// Histogram copies in global memory (u64), indexed by work unit.
constexpr int kGlobalCopies = 64;
// Largest number of output slots (nbins <= 256 -> nbins + 2 slots).
constexpr int kMaxSlots = 258;

// Table entry encoding.  A cell of the squared-chord (FP32) or 1 - d (FP64)
// axis maps to:
//   0 .. kMaxSlots-1   the slot, certain for every value in the cell;
//   kMedium | k        exactly one edge k is undecided inside the cell;
//   kMulti             several edges are undecided: use the exact rule.
// One-byte tables use 0x80 | k and 0xFF instead (slots and k below 0x7F).
constexpr uint16_t kMedium = 0x8000;
constexpr uint16_t kMulti = 0xFFFF;
constexpr int kMaxSlots8 = 127;
// Cell entries of the FP32 tiles: slot * bytes between histogram rows (a
// power of two, at least 16), flags below.
constexpr uint32_t kCellOpen = 1;    // an edge lies in the cell, between the slot and the next
constexpr uint32_t kCellMulti = 2;   // several edges (kCellOpen is set too)

// FP32 tiles: the edge a tile's pairs are compared with, the one nearest to
// its column's distance q from the rows' mean: of the column's slot (lower end
// and width as in PairArgs::tile_slots) the upper edge above the slot's middle
// and the lower one up to it.  The first slot has no lower edge and the last
// no upper one, and both may have no width (a first edge whose band reaches 0,
// with a column at the mean itself; a last edge out of reach), so the number
// is clamped here, once for all that it is used for.
TPCF_HD uint32_t nearest_edge(uint32_t slot, float q, float lower, float width, uint32_t nedges) {
    const int32_t k = q > fmaf(0.5f, width, lower) ? (int32_t)slot : (int32_t)slot - 1, last = (int32_t)nedges - 1;
#ifdef __HIP_DEVICE_COMPILE__
    int32_t r;      // (one instruction where the compiler takes two or three)
    asm("v_med3_i32 %0, %1, 0, %2" : "=v"(r) : "v"(k), "v"(last));
    return (uint32_t)r;
#else
    return (uint32_t)std::min(std::max(k, 0), last);
#endif
}

// One work unit: the row tile starting at i0 with valid rows [row_lo, i1),
// against columns j in [j0, j1) of job `job` (col_lo == j0, kept for the
// plan's bookkeeping).  A unit needs per-pair masking when its valid rows do
// not fill the tile or, for auto-pairs, when its columns overlap its rows
// (the j <= i diagonal).
// reg_a / reg_b: jackknife regions of the unit's rows and columns (-1: none).
struct Unit {
    int32_t i0, i1, j0, j1;
    int32_t job, row_lo, col_lo, reg_a;
    int32_t reg_b, pad0, pad1, pad2;
};

// One counting job of a launch: catalogs A (rows i) and B (columns j) as
// structures of arrays, the pair kind, and where its histogram goes.
struct JobDev {
    const float *ax32, *ay32, *az32;
    const float *bx32, *by32, *bz32;
    const double *ax64, *ay64, *az64;
    const double *bx64, *by64, *bz64;
    // Bounding caps of the column catalog's aligned 64-point groups (stored
    // order): centre x, y, z and an upper bound of the angular radius (3-D:
    // the points' mean and the largest distance from it); null unless
    // pruning is on.
    const double *bcaps;
    unsigned long long *hist;    // kGlobalCopies x nslots, zeroed before
    // jackknife regions: nreg x kGlobalCopies x nslots, zeroed before; the
    // histogram of a unit also goes to its rows' and columns' regions (once
    // when they coincide).  Null without regions.
    unsigned long long *touch;
    const int *cancel;           // host-visible flag (non-zero: skip the rest), or null
    int32_t auto_pairs;          // 1: DD/RR (count j > i only), 0: DR
    int32_t na, nb;              // catalog sizes
    int32_t pad;
};

struct PairArgs {
    const JobDev *jobs;          // device job table, or null: every unit belongs to job0
    JobDev job0;                 // the job of a single-job launch (passed by value)
    const Unit *units;           // device, or null: units of `grid`
    UnitGrid grid;
    int32_t n_units;
    // Work queues: item i is wavefront part i % kWaves of unit i / kWaves;
    // each wavefront takes the item of its own number, then one at a time by
    // atomic adds on kQueues counters (zeroed before the launch).
    unsigned int *queue;

    // Cell table (device, copied into LDS by every block).
    const void *lut;
    int32_t lut_cells;           // c_hi - c_lo + 1
    int32_t lut_entry_bytes;     // 1 or 2
    int32_t lut_shift;           // cell = key >> shift
    int32_t lut_lo, lut_hi;      // clamp range of cells
    // FP64 path, pairs certainly beyond the last edge: the high word of e =
    // 1 - d above beyond_key as signed integers (e > E_last), or with
    // beyond_dot, that of d below it (d < D_last).
    uint32_t beyond_key;
    int32_t beyond_dot;
    // FP32 tiles: every squared distance (cell table, bands) is scaled by q_scale^2 = 2^q_exp2, q_scale the power of two that brings the
    // coordinates into f16's range.  q_small: steps with a column below it
    // from the rows' mean are counted as chord steps (-inf: none).
    // tile_slots (nslots): lower end and width of every slot; tile_edges
    // (nedges): qhi, qhi - qlo, and how far below and above it x = q - qhi
    // may reach without meeting another edge's band.  Null on other paths.
    float q_scale;
    int32_t q_exp2;
    float q_small;
    const float2 *tile_slots;
    const float4 *tile_edges;

    // Exact tile pruning: 1 = a wavefront bins a whole aligned 64-column
    // block at once when the bounding caps put every pair of the block
    // strictly inside one slot.
    int32_t prune;

    // 0: angles on the sky (dot products against D_k); 1: 3-D distances
    // (squared distances of Cartesian points, D_k = -S_k, E_k = S_k).
    int32_t metric;
    // 3-D pruning: absolute widening of the distance interval of a block
    // (covers the FP32 copies of the rows, 2^-22 times the largest norm).
    double prune_margin;
    // Angular pruning: bound on | |v|^2 - 1 | of the catalogs' stored
    // vectors (the rule's dot product is |v_i| |v_j| cos(phi), not cos(phi)).
    double prune_delta;

    // Edge thresholds (device).
    const float *qlo, *qhi;      // FP32 chord^2 bands, nedges each
    const double *E;             // fl(1 - D_k), nedges
    const double *D;             // D_k, nedges
    int32_t nedges;              // nbins + 1
    int32_t nslots;              // nbins + 2

    // Per-wave LDS histogram copies (layout [slot][copy]).
    int32_t hist_copies;         // 32, 16, 8 or 4
    int32_t rows_per_lane;       // 2 or 4 (FP32 without pruning: or 1): a unit spans kWaves * 64 * rows_per_lane rows
    int32_t blocks_per_cu;       // grid = CUs x this (0: the blocks that fit at once)

    unsigned long long *stats;   // kStatCopies times kStats words: [two-slot steps, flagged, exact, skipped
                                 //  units, rare-path steps, steps counted beyond the last
                                 //  edge, one-slot steps, pairs binned by pruned blocks,
                                 //  angular FP32 steps that formed the chord]
};

// LDS bytes per edge: for the tiles D_k, the FP32 chord band (qlo_k, qhi_k)
// and the tiles' edge entry; FP64 launches use 16 of them (D_k, fl(1 - D_k)).
constexpr int kEdgeLdsBytes = 8 + 8 + 8 + 8;

// LDS bytes of the histograms (with the discard row) and edge thresholds.
inline int aux_lds_bytes(int nslots, int hist_copies, int nedges) {
    int hist = kWaves * (nslots + 1) * hist_copies * 4;
    int thr = nedges * kEdgeLdsBytes;
    return hist + thr;
}

// LDS bytes used by one block for the given table sizes.
inline int lds_bytes(int nslots, int hist_copies, int lut_cells, int lut_entry_bytes, int nedges) {
    return (((lut_cells * lut_entry_bytes) + 15) & ~15) + aux_lds_bytes(nslots, hist_copies, nedges);
}

// What FP32 tiles hold besides: the slot table and every wavefront's buffer
// of 64 columns.
constexpr int kStageWaveBytes = 3 * 64 * 4;
inline int tile_lds_bytes(int nslots) { return nslots * 8 + kWaves * kStageWaveBytes; }

// Margin (radians) of the geometric angle interval of the pruning test:
// covers the FP32 copies of the rows (directions move by <= 1.2e-7 rad) and
// the rounding of the caps' arithmetic (<= ~3e-8 rad, acos near 1 included).
constexpr double kPruneMargin = 1e-6;
// Absolute slack of the pruning test's dot-product interval: the rule's own
// rounding (gamma_3 (1 + delta) < 3.4e-16) and that of the interval
// arithmetic (a few units of 2^-53).
constexpr double kPruneDotSlack = 2e-15;

}  // namespace tpcf

// Size of the fixed per-device work area of tpcf_count_noalloc (histogram
// copies, work queues, output slots, edge and cell tables, and the
// work-unit list).
constexpr size_t kScratchBytes = size_t(16) << 20;

// Launchers implemented in kernels.hip.
extern "C" {
// Look up (once per device, with that device current) the device address of
// the fixed work area; 0 or a hipError_t.
int tpcf_scratch_init(int device);
// The address found by tpcf_scratch_init for this device, or null.
void *tpcf_scratch_ptr(int device);
int tpcf_launch_pairs(const tpcf::PairArgs *args, int precision, void *stream);
int tpcf_launch_zero_u64(unsigned long long *p, int64_t n, void *stream);
// Sum the kGlobalCopies copies of each of njobs histograms (contiguous,
// njobs x kGlobalCopies x nslots) into out (njobs x nslots).
int tpcf_launch_reduce_copies(unsigned long long *copies, int32_t nslots, int32_t njobs,
                              unsigned long long *out, void *stream);
// The same for one histogram, leaving its copies and the queue_words after
// them zero.
int tpcf_launch_reduce_clear(unsigned long long *copies, int32_t nslots, int32_t queue_words,
                             unsigned long long *out, void *stream);
// FP32 copies of an FP64 SoA catalog, or (given32 non-null) a check that
// given32 holds them; check_out[0] receives the largest | |v|^2 - 1 | (bits
// of a double, +inf for a non-finite value), check_out[1] a non-zero value
// if a given copy differs.  check_out is zeroed by the caller.
int tpcf_launch_to_float(const double *xyz64, int64_t n, float *xyz32, const float *given32,
                         unsigned long long *check_out, void *stream);
// Bounding caps of the aligned 64-point groups of an FP64 SoA catalog
// (see JobDev::bcaps): 4 doubles per group; metric 1 (3-D): bounding balls.
int tpcf_launch_caps64(const double *xyz64, int64_t n, double *caps, int metric, void *stream);
}
