// Pair-counting kernels for gfx950 (MI355X).
//
// The method (paper, Section 3): form the angle of every pair of objects from
// the dot product of their unit vectors, and histogram it with atomic
// updates of per-block partial histograms in on-chip memory that are later
// combined in one histogram in global memory.
//
// gfx950 design:
//   * FP32 launches form the squared distances of 32 x 32 pairs at a time on
//     the matrix cores and bin whole tiles (see "FP32 tiles on the matrix
//     cores" below); the points below are the FP64 vector path;
//   * one work unit = a tile of rows i (four wavefronts, each holding P = 2
//     or 4 points per lane in registers) against a range of columns
//     j; every wavefront walks the same j range, reading each j through the
//     scalar unit (the address is uniform), so no LDS staging of j is needed;
//   * a pair is classified with one table lookup in LDS: the key is the top
//     bits of e = fl64(1 - d); a cell whose whole range lies between two
//     edges gives the slot directly, a cell that straddles one edge is
//     settled by one threshold comparison, and anything closer is re-decided
//     with the exact rule d <= D_k;
//   * every wavefront owns a private LDS histogram, layout [slot][copy] with
//     copy = lane mod copies, updated with ds_add_u32;
//   * a wavefront sums its histogram when its items go to another job (and
//     at the end) and adds it with 64-bit atomics into one of kGlobalCopies
//     global copies, which a final kernel reduces into the output slots.
//
// The whole file is compiled with -ffp-contract=off: the FP64 dot product is
// evaluated unfused and left to right exactly like the counting rule; the
// FP32 chord^2 uses explicit fmaf, which the error band accounts for.
#include <hip/hip_runtime.h>

#include <mutex>

#include "internal.h"

using namespace tpcf;

namespace {

// Columns per step of the FP64 vector path (each lane evaluates P x this many
// pairs between two wavefront-wide tests): 12 % slower at 4 than at 2 on the
// octant workload, for the registers.
constexpr int kColsPerStepF64 = 2;

typedef __attribute__((address_space(3))) uint32_t lds_u32;
typedef __attribute__((address_space(3))) uint16_t lds_u16;
typedef __attribute__((address_space(3))) uint8_t lds_u8;

// Column coordinates are read through the constant address space: every lane
// of a wavefront reads the same j, so these become scalar loads into SGPRs.
typedef const __attribute__((address_space(4))) double *cdouble_p;
typedef const __attribute__((address_space(4))) uint32_t *cword_p;

// Unit and job descriptors are read-only and wavefront-uniform as well: copy
// them word by word through the constant address space (scalar loads).
template <typename T>
__device__ __forceinline__ T load_uniform(const T *p) {
    static_assert(sizeof(T) % 4 == 0, "descriptor size");
    T out;
    cword_p src = (cword_p)p;
    uint32_t *dst = reinterpret_cast<uint32_t *>(&out);
#pragma unroll
    for (int w = 0; w < (int)(sizeof(T) / 4); ++w)
        dst[w] = src[w];
    return out;
}

// Clamp into [lo, hi] in one instruction (all operands in VGPRs: gfx9 VOP3
// reads at most one SGPR, which keeps the compiler from forming v_med3).
__device__ __forceinline__ int32_t med3_i32(int32_t x, int32_t lo, int32_t hi) {
    int32_t r;
    asm("v_med3_i32 %0, %1, %2, %3" : "=v"(r) : "v"(x), "v"(lo), "v"(hi));
    return r;
}

// Copy a wavefront-uniform value into a VGPR once, so loops do not
// re-materialise it for every VOP3 that needs a VGPR operand.
__device__ __forceinline__ uint32_t to_vgpr(uint32_t x) {
    uint32_t r;
    asm("v_mov_b32 %0, %1" : "=v"(r) : "s"(x));
    return r;
}

// LDS access by 32-bit byte address.
template <bool LUT8>
__device__ __forceinline__ uint32_t lds_read_entry(uint32_t addr) {
    if (LUT8)
        return *(const lds_u8 *)(uintptr_t)addr;
    return *(const lds_u16 *)(uintptr_t)addr;
}

__device__ __forceinline__ void lds_add(uint32_t addr, uint32_t v) {
    __hip_atomic_fetch_add((lds_u32 *)(uintptr_t)addr, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// True when `pred` holds on every lane of the (fully active) wavefront.
__device__ __forceinline__ bool wave_all(bool pred) {
    return __builtin_amdgcn_ballot_w64(pred) == ~0ull;
}

// Balanced reductions of the JN x P values of a step (depth ~log3 instead
// of a chain of JN * P dependent instructions).
template <typename T, typename F, int N>
__device__ __forceinline__ T tree_reduce(const T (&v)[N], F f) {
    if constexpr (N == 1) {
        return v[0];
    } else if constexpr (N == 2) {
        return f(v[0], v[1]);
    } else {
        constexpr int M = (N + 2) / 3;
        T w[M];
#pragma unroll
        for (int i = 0; i < M; ++i) {
            T x = v[3 * i];
            if (3 * i + 1 < N)
                x = f(x, v[3 * i + 1]);
            if (3 * i + 2 < N)
                x = f(x, v[3 * i + 2]);
            w[i] = x;
        }
        return tree_reduce<T, F, M>(w, f);
    }
}

__device__ __forceinline__ void lds_inc(uint32_t addr) {
    __hip_atomic_fetch_add((lds_u32 *)(uintptr_t)addr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Cell entry codes: a slot (certain for the whole cell), flag | k (edge k
// undecided), or flag | kmask (several edges undecided).  Every test of an
// entry takes the flag bit from a register (Consts::flag): with literal masks
// the compiler narrows the tests to 8 or 16 bits and then spends an extra
// instruction per entry to widen the loaded value again.
template <bool LUT8>
struct Code {
    static constexpr uint32_t flag = LUT8 ? 0x80u : 0x8000u;
    static constexpr uint32_t kmask = LUT8 ? 0x7Fu : 0x7FFFu;
};

// Number of k with d <= D[k]; D is non-increasing in k.
__device__ __forceinline__ uint32_t count_le(double d, const double *D, int n) {
    int lo = 0, hi = n;
    while (lo < hi) {
        int mid = (lo + hi) >> 1;
        if (d <= D[mid])
            lo = mid + 1;
        else
            hi = mid;
    }
    return (uint32_t)lo;
}

// FP64 dot product of the counting rule: (x_i x_j + y_i y_j) + z_i z_j with
// every operation rounded (contraction is off for this file).
__device__ __forceinline__ double exact_dot(double xi, double yi, double zi,
                                            double xj, double yj, double zj) {
    double t = xi * xj;
    double u = yi * yj;
    double s = t + u;
    double v = zi * zj;
    return s + v;
}

// 3-D: squared distance of the counting rule, (dx^2 + dy^2) + dz^2 of the
// FP64 coordinate differences, every operation rounded.
__device__ __forceinline__ double exact_d2(double xi, double yi, double zi,
                                           double xj, double yj, double zj) {
    double dx = xi - xj;
    double dy = yi - yj;
    double dz = zi - zj;
    double t = dx * dx;
    double u = dy * dy;
    double s = t + u;
    double v = dz * dz;
    return s + v;
}

// The value the thresholds D_k are compared with (past edge k when
// value <= D_k): the dot product for angles, minus the squared distance in
// 3-D (where D_k = -S_k).
template <bool M3>
__device__ __forceinline__ double rule_value(double xi, double yi, double zi,
                                             double xj, double yj, double zj) {
    return M3 ? -exact_d2(xi, yi, zi, xj, yj, zj) : exact_dot(xi, yi, zi, xj, yj, zj);
}

struct Smem {
    uint32_t *hist;      // kWaves x (nslots + 1) x copies
    double *D;
    double *E;
    float2 *qband;       // FP32 band (qlo_k, qhi_k), one 8-byte read per edge
    float2 *slots;       // FP32 tiles: lower end and width of every slot
    uint32_t stage_addr; // FP32 tiles: LDS byte address of the wavefronts' column buffers
    float4 *edges;       // FP32 tiles: qhi, qhi - qlo, room below and above every edge
    unsigned char *lut;
    uint32_t hist_addr;  // LDS byte address of hist
    uint32_t lut_addr;   // LDS byte address of lut
};

// LDS layout: the cell table, then the histograms and the edge thresholds.
template <bool TILES>
__device__ __forceinline__ Smem carve(unsigned char *base, const PairArgs &a) {
    Smem s = {};
    const int aux = (a.lut_cells * a.lut_entry_bytes + 15) & ~15;
    int hist_words = kWaves * (a.nslots + 1) * a.hist_copies;
    s.lut = base;
    s.hist = reinterpret_cast<uint32_t *>(base + aux);
    unsigned char *edges = base + aux + hist_words * 4;     // 16-aligned
    if (TILES) {
        s.edges = reinterpret_cast<float4 *>(edges);
        s.D = reinterpret_cast<double *>(s.edges + a.nedges);
        s.qband = reinterpret_cast<float2 *>(s.D + a.nedges);
        s.slots = s.qband + a.nedges;
        s.stage_addr = (uint32_t)(uintptr_t)(lds_u32 *)(s.slots + a.nslots);
    } else {
        s.D = reinterpret_cast<double *>(edges);
        s.E = s.D + a.nedges;
    }
    s.hist_addr = (uint32_t)(uintptr_t)(lds_u32 *)s.hist;
    s.lut_addr = (uint32_t)(uintptr_t)(lds_u8 *)s.lut;
    return s;
}

__device__ __forceinline__ double wave_max_d(double v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
        v = fmax(v, __shfl_xor(v, off, kWaveSize));
    return v;
}

__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
        v += __shfl_xor(v, off, kWaveSize);
    return v;
}

// Sum one wavefront's LDS histogram into a global copy and clear it; with
// region copies (r0, r1 non-null) the sums also go there.
__device__ void flush_wave(const PairArgs &a, const Smem &s, unsigned long long *hist, unsigned long long *r0,
                           unsigned long long *r1, int wave, int lane, int copy) {
    const int C = a.hist_copies;
    uint32_t *h = s.hist + wave * (a.nslots + 1) * C;
    const size_t off = (size_t)copy * a.nslots;
    for (int s0 = 0; s0 < a.nslots; s0 += kWaveSize) {
        int slot = s0 + lane;
        if (slot < a.nslots) {
            uint32_t acc = 0;
            uint32_t *row = h + slot * C;
            // skewed walk over the copies: lanes of a half-wave hit distinct banks
            for (int c = 0; c < C; ++c) {
                int cc = (c + lane) & (C - 1);
                acc += row[cc];
                row[cc] = 0;
            }
            if (acc) {
                atomicAdd(&hist[off + slot], (unsigned long long)acc);
                if (r0)
                    atomicAdd(&r0[off + slot], (unsigned long long)acc);
                if (r1)
                    atomicAdd(&r1[off + slot], (unsigned long long)acc);
            }
        }
    }
}

// A flagged entry: edge k alone is undecided in the cell (e against E_k, a tie
// by the rule), or several are (the rule counts them).
template <bool LUT8>
__device__ __forceinline__ uint32_t resolve_fp64(uint32_t ent, uint32_t flag, double e, double d,
                                                 const Smem &s, const PairArgs &a,
                                                 uint32_t &n_exact) {
    if (ent != (flag | Code<LUT8>::kmask)) {
        int k = (int)(ent ^ flag);
        double Ek = s.E[k];
        if (e > Ek)
            return (uint32_t)(k + 1);
        if (e < Ek)
            return (uint32_t)k;
        ++n_exact;
        return (uint32_t)k + (d <= s.D[k] ? 1u : 0u);
    }
    ++n_exact;
    return count_le(d, s.D, a.nedges);
}

// Work statistics of one lane: pairs that left the table path, pairs decided
// by the exact FP64 rule, and (wavefront-uniform) steps that took the rare path.
struct Counters {
    uint32_t flag = 0, exact = 0, rare = 0;
    uint32_t beyond = 0;        // this lane's pairs counted beyond the last edge (per unit)
    // Step kinds of the current column range on the vector paths, 16 bits
    // each (wavefront-uniform, kept in scalar registers): steps beyond the
    // last edge, in one slot, in two slots; folded into the totals below
    // after every range of at most kFoldCols columns.
    uint64_t steps = 0;
    uint32_t beyond_steps = 0, one_slot_steps = 0, two_slot_steps = 0, chord_steps = 0;
    uint32_t pruned_blocks = 0;     // wavefront blocks (P x 64 rows x 64 columns) binned whole (uniform)

    __device__ __forceinline__ void fold() {
        beyond_steps += (uint32_t)(steps & 0xFFFF);
        one_slot_steps += (uint32_t)((steps >> 16) & 0xFFFF);
        two_slot_steps += (uint32_t)((steps >> 32) & 0xFFFF);
        steps = 0;
    }
};

// Longest column range one call of the column loops covers: at most
// kFoldCols / 2 steps, below the 16-bit step fields of Counters.
constexpr int kFoldCols = 65536;

// How a wavefront step was binned (wavefront-uniform).  A step beyond the
// last edge adds nothing to the histograms: the caller counts its pairs in
// the lane's register.
enum : uint32_t { kBeyond = 0, kOneSlot = 1, kTwoSlot = 2, kLookup = 3 };

// Per-step bookkeeping, done once after the step whichever way it went (so
// the counters are not carried through the step's branches).  The step
// functions' codes are wavefront-uniform, but the compiler cannot tell
// (their paths hold per-lane branches), so the callers pass them through
// readfirstlane to keep the code and the branches on it scalar.
template <uint32_t N>
__device__ __forceinline__ void account(uint32_t code, Counters &cnt) {
    cnt.beyond += code == kBeyond ? N : 0u;
    cnt.steps += code <= kTwoSlot ? (uint64_t)1 << (16 * code) : 0;
}

// Loop constants of one wavefront.
struct Consts {
    uint32_t shift;
    uint32_t clo, chi;      // clamp range (VGPR copies)
    uint32_t lutbias;       // LDS address of cell c is c * entry_bytes + lutbias
    uint32_t rowstep;       // bytes between slots of the histogram
    uint32_t rowlog;        // its logarithm
    uint32_t lanebase;      // LDS address of this lane's copy of slot 0
    uint32_t flag;          // flag bit of the cell entries (VGPR copy)
    uint32_t beyond;        // PairArgs::beyond_key (VGPR copy)
    bool by_dot;            // PairArgs::beyond_dot
};

// LDS address of the cell-table entry of an FP64 key (the high word of e;
// arithmetic shift, so e < 0 lands in the bottom cell).
template <bool LUT8>
__device__ __forceinline__ uint32_t addr64(int32_t hi, const Consts &k) {
    const int32_t c = med3_i32(hi >> (int)k.shift, (int32_t)k.clo, (int32_t)k.chi);
    return (uint32_t)c * (LUT8 ? 1u : 2u) + k.lutbias;
}

// Slot range of a lane's pairs.  A cell entry bounds the slots of its keys: a
// certain slot s gives [s, s], edge k undecided gives [k, k+1] (a cell with
// several undecided edges gives [kmask, kmask+1], which no test below
// accepts).  Slots never decrease as the key grows (keys below the table
// share its bottom cell), so the entries of a lane's smallest and largest key
// bound the slots of all its pairs: lo = the lower end of the first, and
// span = the upper end of the second minus lo.
template <bool LUT8>
__device__ __forceinline__ void slot_range(uint32_t e_lo, uint32_t e_hi, uint32_t &lo, uint32_t &span) {
    constexpr uint32_t m = Code<LUT8>::kmask, sh = LUT8 ? 7 : 15;
    lo = e_lo & m;
    span = (e_hi & m) + (e_hi >> sh) - lo;
}

// One slot for all of a lane's pairs (span 0).  When that holds on every lane
// the step adds its pairs with one LDS atomic per lane instead of a lookup and
// an atomic per pair.  A lane's rows (and a wavefront's) are consecutive in
// the Morton order, so at angles large against their extent this is common.
__device__ __forceinline__ bool one_slot_step(uint32_t lo, uint32_t span, uint32_t n, const Consts &k,
                                              Counters &cnt) {
    if (!wave_all(span == 0))
        return false;
    lds_add(__umul24(lo, k.rowstep) + k.lanebase, n);
    return true;
}

// Two adjacent slots [lo, lo+1] (or one) for all of a lane's pairs, on every
// lane: then each pair needs one comparison with edge lo's threshold instead
// of a table lookup, and the step adds its pairs with two LDS atomics per
// lane.
template <bool LUT8>
__device__ __forceinline__ bool two_slot_range(uint32_t lo, uint32_t span) {
    return (__builtin_amdgcn_ballot_w64(span <= 1u) & __builtin_amdgcn_ballot_w64(lo != Code<LUT8>::kmask)) == ~0ull;
}

__device__ __forceinline__ void two_slot_add(uint32_t base, uint32_t n, uint32_t n_up, const Consts &k,
                                             Counters &cnt) {
    // both adds on every lane (a lane with one slot adds 0 to the next row,
    // at most the discard row): no per-lane branch, so the step's outcome
    // stays wavefront-uniform for the compiler
    const uint32_t addr = __umul24(base, k.rowstep) + k.lanebase;
    lds_add(addr, n - n_up);
    lds_add(addr + k.rowstep, n_up);
}

// ---------------------------------------------------------------------------
// Exact tile pruning.  A bounding cap (unit centre c, angular radius rho) of
// the wavefront's rows and one of an aligned 64-column block bound the
// geometric angle phi (between the normalised directions) of every pair of
// the block to [acos(c_r . c_b) - rho_r - rho_b, acos(c_r . c_b) + rho_r +
// rho_b], widened by kPruneMargin (the FP32 row copies and the cap
// arithmetic).  The counting rule does not see phi but the FP64 dot product
// of the stored vectors, whose squared norms deviate from 1 by up to delta:
// d = |v_i| |v_j| cos(phi) + err with |v_i| |v_j| in [1 - delta, 1 + delta]
// and |err| <= kPruneDotSlack (the rule's rounding).  So every pair's d lies
// in [lo - delta |lo| - slack, hi + delta |hi| + slack] for any bounds
// lo <= cos(phi) <= hi over the block (dot_range forms them without
// trigonometric functions); when no threshold D_k falls inside that interval
// every pair passes the same edges, and the wavefront adds the block's pairs
// to that slot without evaluating them.

__device__ __forceinline__ double wave_sum_d(double v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
        v += __shfl_xor(v, off, kWaveSize);
    return v;
}

__device__ __forceinline__ double wave_min_d(double v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
        v = fmin(v, __shfl_xor(v, off, kWaveSize));
    return v;
}

struct Cap {
    double x, y, z, rho;
};

// A wavefront-uniform double moved to scalar registers (lane 0's value).
__device__ __forceinline__ double uniform_d(double v) {
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    // readfirstlane returns a signed int: take its 32 bits without sign extension
    const uint64_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)b);
    const uint64_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
    return __longlong_as_double((long long)((hi << 32) | lo));
}

__device__ __forceinline__ Cap uniform_cap(const Cap &c) {
    return Cap{uniform_d(c.x), uniform_d(c.y), uniform_d(c.z), uniform_d(c.rho)};
}

// Cap of the points (x, y, z) held by the lanes (every lane contributes n
// points; duplicates are harmless).  Identical on every lane.
template <int N>
__device__ __forceinline__ Cap cap_of(const double (&x)[N], const double (&y)[N], const double (&z)[N]) {
    double sx = 0.0, sy = 0.0, sz = 0.0;
#pragma unroll
    for (int p = 0; p < N; ++p) {
        sx += x[p];
        sy += y[p];
        sz += z[p];
    }
    sx = wave_sum_d(sx);
    sy = wave_sum_d(sy);
    sz = wave_sum_d(sz);
    const double norm = sqrt(sx * sx + sy * sy + sz * sz);
    Cap c;
    if (!(norm > 1e-3)) {       // points spread over the sphere: no useful cap
        c.x = 1.0;
        c.y = c.z = 0.0;
        c.rho = M_PI;
        return c;
    }
    c.x = sx / norm;
    c.y = sy / norm;
    c.z = sz / norm;
    double m = 1.0;
#pragma unroll
    for (int p = 0; p < N; ++p) {
        const double len = sqrt(x[p] * x[p] + y[p] * y[p] + z[p] * z[p]);
        m = fmin(m, (c.x * x[p] + c.y * y[p] + c.z * z[p]) / len);
    }
    m = wave_min_d(m);
    c.rho = acos(fmin(fmax(m, -1.0), 1.0)) + 1e-12;
    return c;
}

// Bounds of the rule's value over every pair between the row cap and a column
// block's cap (delta bounds the catalogs' | |v|^2 - 1 |).  With
// c = cos(theta_c) the dot product of the two centres, sn an upper bound of
// sin(theta_c) and rho the summed radii, every pair's geometric angle is
// theta_c + t with |t| <= rho, and
// cos(theta_c + t) = c cos t - sin(theta_c) sin t lies within
// [c - sn rho - max(c, 0) rho^2 / 2, c + sn rho + max(-c, 0) rho^2 / 2]
// (1 - t^2 / 2 <= cos t <= 1, |sin t| <= |t|).  No trigonometric function is
// evaluated; the margin in rho (1e-6 rad) widens the interval by at least
// sn 1e-6 > 6e-14, far above the rounding of this arithmetic.
__device__ __forceinline__ void dot_range(const Cap &r, const Cap &b, double delta, double &lo, double &hi) {
    const double c = fmin(fmax(r.x * b.x + r.y * b.y + r.z * b.z, -1.0), 1.0);
    const double rho = r.rho + b.rho + kPruneMargin;
    const double h = 0.5 * rho * rho;
    // an upper bound of the sine: 1 - c^2 formed as (1 - c)(1 + c), plus the
    // rounding of c and of that product
    const double sn = sqrt((1.0 - c) * (1.0 + c) + 4e-15);
    hi = c + sn * rho + fmax(-c, 0.0) * h;
    lo = c - sn * rho - fmax(c, 0.0) * h;
    hi = hi + delta * fabs(hi) + kPruneDotSlack;
    lo = lo - delta * fabs(lo) - kPruneDotSlack;
}

// 3-D: bounding ball of the points held by the lanes (centre = their mean,
// radius = the largest distance from it, widened by 1e-12 relative).
// Identical on every lane.
template <int N>
__device__ __forceinline__ Cap ball_of(const double (&x)[N], const double (&y)[N], const double (&z)[N]) {
    double sx = 0.0, sy = 0.0, sz = 0.0;
#pragma unroll
    for (int p = 0; p < N; ++p) {
        sx += x[p];
        sy += y[p];
        sz += z[p];
    }
    const double inv = 1.0 / (double)(N * kWaveSize);
    Cap c;
    c.x = wave_sum_d(sx) * inv;
    c.y = wave_sum_d(sy) * inv;
    c.z = wave_sum_d(sz) * inv;
    double m = 0.0;
#pragma unroll
    for (int p = 0; p < N; ++p) {
        const double dx = x[p] - c.x, dy = y[p] - c.y, dz = z[p] - c.z;
        m = fmax(m, sqrt(dx * dx + dy * dy + dz * dz));
    }
    c.rho = wave_max_d(m) * (1.0 + 1e-12);
    return c;
}

// 3-D: bounds of the rule's value, minus the squared distance.  The distances
// lie within [|c_r - c_b| -+ (rho_r + rho_b)], widened by margin (the FP32
// copies of the rows, at most 2^-22 R) and by 1e-12 relative (the rule's and
// this arithmetic's rounding, the squares below included; 1e-300 covers
// squares that round to subnormal numbers).
__device__ __forceinline__ void d2_range(const Cap &r, const Cap &b, double margin, double &lo, double &hi) {
    const double dx = r.x - b.x, dy = r.y - b.y, dz = r.z - b.z;
    const double dc = sqrt(dx * dx + dy * dy + dz * dz);
    const double spread = r.rho + b.rho;
    const double w = margin + 1e-12 * (dc + spread);
    const double near = fmax(dc - spread - w, 0.0), far = dc + spread + w;
    hi = -fmax(near * near - 1e-300, 0.0);
    lo = -(far * far) - 1e-300;
}

// Block cap for either metric.
template <bool M3, int N>
__device__ __forceinline__ Cap block_cap(const double (&x)[N], const double (&y)[N], const double (&z)[N]) {
    return uniform_cap(M3 ? ball_of<N>(x, y, z) : cap_of<N>(x, y, z));
}

// Columns one call of prune_blocks covers, from an aligned one on.
constexpr int kPruneCols = 64 * kWaveSize;

// The aligned 64-column blocks of [j0, j1) (64 of them at most), against the
// row cap r of a wavefront with all of its rows: those that lie whole in the
// range, past its masked columns (up to jm), and are proven to hold pairs of one slot only are binned (n pairs
// each); bit b of the result is set for the others.  One lane per block and one binary search
// over the thresholds for both ends of the range: testing the blocks one by
// one, a lane per threshold, took the whole wavefront as long for one block
// as this takes for all of them.
template <bool M3>
__device__ __forceinline__ uint64_t prune_blocks(const Cap &r, const double *bcaps, const Smem &s, const PairArgs &a,
                                                 const Consts &k, int j0, int j1, int jm, uint32_t n, int lane,
                                                 Counters &cnt) {
    const int64_t b = (int64_t)(j0 >> 6) + lane;
    bool one = 64 * b >= max(j0, jm) && 64 * b + 64 <= j1;
    if (one) {
        const double *c = bcaps + 4 * b;
        const Cap bc{c[0], c[1], c[2], c[3]};
        double lo, hi;
        if (M3)
            d2_range(r, bc, a.prune_margin, lo, hi);
        else
            dot_range(r, bc, a.prune_delta, lo, hi);
        // pairs with the largest value pass the fewest edges
        const uint32_t slot = count_le(hi, s.D, a.nedges);
        one = slot == (uint32_t)a.nedges || lo > s.D[slot];
        if (one && slot == (uint32_t)(a.nslots - 1))
            cnt.beyond += n;
        else if (one)
            lds_add(__umul24(slot, k.rowstep) + k.lanebase, n);
    }
    const uint64_t done = __builtin_amdgcn_ballot_w64(one);
    cnt.pruned_blocks += (uint32_t)__builtin_popcountll(done);
    return __builtin_amdgcn_ballot_w64(64 * b < j1) & ~done;
}

// Row p of a wavefront lane whose rows start at ib: lane L holds the P
// consecutive rows ib + P L ... ib + P L + P - 1.  Rows are stored in Morton
// order, so a lane's rows lie close together and its pairs of a step span a
// narrow range of angles: more lanes fall in one slot, or in two adjacent
// ones, than with rows 64 apart.
template <int P>
__device__ __forceinline__ int row_of(int ib, int lane, int p) {
    return ib + lane * P + p;
}

// One step: JN columns against the P rows of every lane.  All JN * P table
// lookups are issued first; one test sends the wavefront to the rare path if
// any lane needs it; then the JN * P histogram increments follow.
template <bool LUT8, bool MASKED, int P, int JN, bool M3, bool ONE>
__device__ __forceinline__ uint32_t step_fp64(const PairArgs &a, const JobDev &jb, const Smem &s, const Consts &k,
                                          const double (&xi)[P], const double (&yi)[P],
                                          const double (&zi)[P], const int (&ii)[P], int ie,
                                          int j, cdouble_p bx, cdouble_p by, cdouble_p bz,
                                          Counters &cnt) {
    double xj[JN], yj[JN], zj[JN];
#pragma unroll
    for (int t = 0; t < JN; ++t) {
        xj[t] = bx[j + t];
        yj[t] = by[j + t];
        zj[t] = bz[j + t];
    }
    // e: the table key's value (1 - d, or r^2 in 3-D); the rule's value d
    // itself is formed again, with the same operations, in the rare path
    double e[JN][P];
    uint32_t ent[JN][P];
#pragma unroll
    for (int t = 0; t < JN; ++t) {
#pragma unroll
        for (int p = 0; p < P; ++p) {
            if (M3)
                e[t][p] = exact_d2(xi[p], yi[p], zi[p], xj[t], yj[t], zj[t]);
            else
                e[t][p] = exact_dot(xi[p], yi[p], zi[p], xj[t], yj[t], zj[t]);
        }
    }
    // a last edge below 90 degrees (D_last > 0): the high word of d below that
    // of D_last implies d < D_last, also for negative d, and steps beyond the
    // edge (61 % on the octant) need no 1 - d, one of their seven operations
    // a pair
    const bool by_dot = !M3 && k.by_dot;
    if (!MASKED && by_dot) {
        int32_t m = __double2hiint(e[0][0]);
#pragma unroll
        for (int t = 0; t < JN; ++t)
#pragma unroll
            for (int p = 0; p < P; ++p)
                m = max(m, __double2hiint(e[t][p]));
        if (wave_all(m < (int32_t)k.beyond))
            return kBeyond;
    }
    if (!M3) {
#pragma unroll
        for (int t = 0; t < JN; ++t)
#pragma unroll
            for (int p = 0; p < P; ++p)
                e[t][p] = 1.0 - e[t][p];
    }
    if (!MASKED) {
        // high word of e above that of E_last implies e > E_last for every pair
        int32_t m = __double2hiint(e[0][0]);
#pragma unroll
        for (int t = 0; t < JN; ++t)
#pragma unroll
            for (int p = 0; p < P; ++p)
                m = min(m, __double2hiint(e[t][p]));
        if (!by_dot && wave_all(m > (int32_t)k.beyond)) {
            return kBeyond;
        }
        if constexpr (ONE) {
            // every pair of the step in one slot (as on the FP32 path)
            int32_t mx = __double2hiint(e[0][0]);
#pragma unroll
            for (int t = 0; t < JN; ++t)
#pragma unroll
                for (int p = 0; p < P; ++p)
                    mx = max(mx, __double2hiint(e[t][p]));
            uint32_t base, span;
            slot_range<LUT8>(lds_read_entry<LUT8>(addr64<LUT8>(m, k)), lds_read_entry<LUT8>(addr64<LUT8>(mx, k)),
                             base, span);
            if (one_slot_step(base, span, JN * P, k, cnt))
                return kOneSlot;
            if (two_slot_range<LUT8>(base, span)) {
                // past edge `base` when e > E_base, not past it when e < E_base,
                // and the exact rule decides e == E_base (as in resolve_fp64);
                // lanes with one slot compare with +inf
                const double thr = span ? s.E[min(base, (uint32_t)(a.nedges - 1))] : __builtin_huge_val();
                // x = fl(e - thr) has the sign of the comparison and is +0
                // only for a tie; a high word of 0 (a tie, or a subnormal x)
                // goes to the lookup
                uint32_t n_below = 0, least = ~0u;
#pragma unroll
                for (int t = 0; t < JN; ++t)
#pragma unroll
                    for (int p = 0; p < P; ++p) {
                        const uint32_t x = (uint32_t)__double2hiint(e[t][p] - thr);
                        n_below += x >> 31;
                        least = min(least, x);
                    }
                // count before the test, so nothing of it stays live past it
                asm volatile("" : "+v"(n_below), "+v"(least));
                if (!__builtin_amdgcn_ballot_w64(least == 0)) {
                    two_slot_add(base, JN * P, JN * P - n_below, k, cnt);
                    return kTwoSlot;
                }
            }
        }
    }
#pragma unroll
    for (int t = 0; t < JN; ++t) {
#pragma unroll
        for (int p = 0; p < P; ++p) {
            ent[t][p] = lds_read_entry<LUT8>(addr64<LUT8>(__double2hiint(e[t][p]), k));
        }
    }
    uint32_t any = 0;
#pragma unroll
    for (int t = 0; t < JN; ++t)
#pragma unroll
        for (int p = 0; p < P; ++p)
            any |= ent[t][p];
    if (any & k.flag) {
        ++cnt.rare;             // wavefront steps that took the rare path
#pragma unroll
        for (int t = 0; t < JN; ++t)
#pragma unroll
            for (int p = 0; p < P; ++p)
                if (ent[t][p] & k.flag) {
                    ++cnt.flag;
                    const double d = rule_value<M3>(xi[p], yi[p], zi[p], xj[t], yj[t], zj[t]);
                    ent[t][p] = resolve_fp64<LUT8>(ent[t][p], k.flag, e[t][p], d, s, a, cnt.exact);
                }
    }
#pragma unroll
    for (int t = 0; t < JN; ++t)
#pragma unroll
        for (int p = 0; p < P; ++p) {
            uint32_t v = ent[t][p];
            if (MASKED) {
                bool ok = ii[p] < ie && (!jb.auto_pairs || j + t > ii[p]);
                v = ok ? v : (uint32_t)a.nslots;
            }
            lds_inc(__umul24(v, k.rowstep) + k.lanebase);
        }
    return kLookup;
}

// Columns [j0, j1) against the P rows of every lane (FP64 vector path).
template <bool LUT8, bool MASKED, int P, bool M3, bool ONE>
__device__ __forceinline__ void cols_fp64(const PairArgs &a, const JobDev &jb, const Smem &s, const Consts &k,
                                          const double (&xi)[P], const double (&yi)[P],
                                          const double (&zi)[P], const int (&ii)[P], int ie, int j0, int j1,
                                          Counters &cnt) {
    cdouble_p bx = (cdouble_p)jb.bx64;
    cdouble_p by = (cdouble_p)jb.by64;
    cdouble_p bz = (cdouble_p)jb.bz64;
    int j = j0;
    for (; j + kColsPerStepF64 <= j1; j += kColsPerStepF64)
        account<kColsPerStepF64 * P>(__builtin_amdgcn_readfirstlane(step_fp64<LUT8, MASKED, P, kColsPerStepF64, M3, ONE>(
                                         a, jb, s, k, xi, yi, zi, ii, ie, j, bx, by, bz, cnt)),
                                     cnt);
    for (; j < j1; ++j)
        account<P>(__builtin_amdgcn_readfirstlane(
                       step_fp64<LUT8, MASKED, P, 1, M3, false>(a, jb, s, k, xi, yi, zi, ii, ie, j, bx, by, bz, cnt)),
                   cnt);
    cnt.fold();
}

template <bool LUT8, bool MASKED, int P, bool PRUNE, bool M3>
__device__ void rows_fp64(const PairArgs &a, const JobDev &jb, const Smem &s, const Consts &k, int ib, int ie,
                          int j0, int j1, int lane, Counters &cnt) {
    double xi[P], yi[P], zi[P];
    int ii[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        int i = row_of<P>(ib, lane, p);
        ii[p] = i;
        int il = i < ie ? i : ib;
        xi[p] = jb.ax64[il];
        yi[p] = jb.ay64[il];
        zi[p] = jb.az64[il];
    }
    if (PRUNE && !MASKED && jb.bcaps) {
        const Cap rc = block_cap<M3, P>(xi, yi, zi);
        for (int jr = j0, je; jr < j1; jr = je) {
            const int b0 = jr >> 6;
            je = part_end(jr, j1, kPruneCols - (jr & 63));
            uint64_t left = prune_blocks<M3>(rc, jb.bcaps, s, a, k, jr, je, jr, P * 64 * 64, lane, cnt);
            while (left) {      // runs of blocks that are left
                const int f = __builtin_ctzll(left);
                const uint64_t gap = ~(left >> f);
                const int e = f + (gap ? __builtin_ctzll(gap) : 64);
                cols_fp64<LUT8, MASKED, P, M3, true>(a, jb, s, k, xi, yi, zi, ii, ie, max(jr, (b0 + f) << 6),
                                                     min(je, (b0 + e) << 6), cnt);
                left = e < 64 ? left & (~0ull << e) : 0;
            }
        }
        return;
    }
    // (unsigned: the position after the last part may lie beyond 31 bits)
    for (uint32_t jc = (uint32_t)j0; jc < (uint32_t)j1; jc += kFoldCols)
        cols_fp64<LUT8, MASKED, P, M3, true>(a, jb, s, k, xi, yi, zi, ii, ie, (int)jc, part_end((int)jc, j1, kFoldCols),
                                             cnt);
}

// ---------------------------------------------------------------------------
// FP32 tiles on the matrix cores.
//
// A wavefront takes 32 G rows (G groups of 32) and walks its columns 32 at a
// time.  One v_mfma_f32_32x32x16_f16 forms the squared distances of a tile
// of 32 rows x 32 columns,
//     q^ = |b'|^2 + |a'|^2 - 2 a'.b',   a' = S (f_i - c),  b' = S (f_j - c),
// of the FP32 copies f relative to the rows' mean c, scaled by S = 2^e (a
// power of two that keeps every operand within f16's range).  Each FP32
// operand enters as the sum of two f16 values (high and low part, all four
// products of a coordinate are formed), |a'|^2 as two more products with a
// constant, and |b'|^2 as the FP32 accumulator input.  A lane holds one
// column against 16 consecutive rows (rows of a group are dealt to the matrix
// rows so that each half of the wavefront gets 16 consecutive ones), so its
// pairs span a narrow range of distances.
//
// |q^ - S^2 |f_i - f_j|^2| <= e = u (kTileErrN |b'|^2 + kTileErrA rho^2 +
// kTileErr0) with u = 2^-24 and rho the largest |a'| of the wavefront.  The
// chord band [qlo_k, qhi_k) holds for |f_i - f_j|^2 itself, so q^ - e >= qhi_k
// puts a pair past edge k and q^ + e < qlo_k before it.  The threshold that a
// test compares with goes into the accumulator input, so the matrix core
// delivers the difference.  Per 32 columns, cheapest first:
//   1. every lane takes the slot of its column's distance from the rows' mean
//      and forms x = q^ - (L + e) for the slot's lower end L: the lane's pairs
//      of a tile are all in that slot when the largest x, as an unsigned bit
//      pattern (negative values lie above all others), is below the slot's
//      width.  No branch and no LDS access; the overflow slot is one of the
//      slots, with an infinite width (tile_screen);
//   2. tiles that fail take the edge nearest to the column's distance,
//      x = q^ - (qhi + e): the sign of x is the pair's side while |x| stays
//      within the neighbouring edges, and the few pairs that lie within e of
//      the band are settled one by one from FP32 differences and, inside the
//      band, by the FP64 rule (tile_split);
//   3. the rest take the slots between the cells of a lane's smallest and
//      largest distance: a few edges are compared with every pair
//      (tile_count), more send every pair to its own cell (tile_cells); by q^
//      where e is at most 2^-10 of it (kTileFar), else by FP32 differences
//      (tile_diffs: close pairs).
// Tiles with masked pairs (the diagonal, the rows' ends) go to 3.
//
// What bounds it: vector issue.  An instruction costs about 4 cycles of a
// SIMD (2 for plain two-operand adds, moves and shifts), the MFMA 32 cycles
// of the matrix core and about 9 of the vector unit's.  Reducing the 16
// values of a lane takes 8 three-operand maxima, so a tile of stage 1 costs
// at least 10 instructions; the preparation of 64 columns (each lane one,
// dealt to two tiles of 32 with v_permlane32_swap) and the accumulator input
// add 5.  Measured: 1e6 x 2e6 points to 30 deg 408 -> 228 ms a DD+DR+RR step
// against the vector kernel it replaces (chord and FP32 dot product), edges
// to 120 deg (2e5 x 4e5) 30.5 -> 18.4 ms, 200 bins 23.0 -> 15.3 ms, a 3-D
// box of 5e5 x 1e6 112.9 -> 53.3 ms; on pairs all beyond the last edge 28
// Tpairs/s (15 before).  Tried and slower: all decisions in one branchy pass
// (307 ms), 32 columns prepared per pass (252), prefetched columns in
// registers (they were spilled and waited for, 246).

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

union Frag {
    uint32_t d[4];
    half8 h;
};

__device__ __forceinline__ uint32_t pack_f16(_Float16 lo, _Float16 hi) {
    union {
        _Float16 h[2];
        uint32_t u;
    } x;
    x.h[0] = lo;
    x.h[1] = hi;
    return x.u;
}

// v as high and low f16 parts, the low one times m (a power of two).
__device__ __forceinline__ uint32_t split_f16(float v, float m) {
    const _Float16 h = (_Float16)v;
    const _Float16 l = (_Float16)((v - (float)h) * m);
    return pack_f16(h, l);
}

__device__ __forceinline__ uint32_t swap_f16(uint32_t x) { return __builtin_amdgcn_alignbit(x, x, 16); }

// |a'|^2 enters as (h 2^14 + l 2^4) with h + l 2^-10 = |a'|^2 2^-14.
constexpr float kNormScale = 6.103515625e-05f;
constexpr float kNormLow = 1024.0f;

__device__ __forceinline__ float wave_sum_f(float v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
        v += __shfl_xor(v, off, kWaveSize);
    return v;
}

__device__ __forceinline__ float wave_max_f(float v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
        v = fmaxf(v, __shfl_xor(v, off, kWaveSize));
    return v;
}

// A wavefront-uniform float moved to a scalar register.
__device__ __forceinline__ float uniform_f(float v) {
    return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(v)));
}

// Squared distance of the FP32 copies from their differences, times S^2.
__device__ __forceinline__ float diff_q(float xi, float yi, float zi, float xj, float yj, float zj, int exp2) {
    const float dx = xi - xj, dy = yi - yj, dz = zi - zj;
    float v = dx * dx;
    v = __fmaf_rn(dy, dy, v);
    v = __fmaf_rn(dz, dz, v);
    return ldexpf(v, exp2);
}

// Element i of the array that starts at the wavefront-uniform address base +
// at: a scalar base and a 32-bit offset per lane.
template <typename T>
__device__ __forceinline__ T lane_load(const T *base, int64_t at, int i) {
    typedef const __attribute__((address_space(1))) char *gchar_p;
    typedef const __attribute__((address_space(1))) T *g_p;
    return *(g_p)((gchar_p)(base + at) + (uint32_t)i * (uint32_t)sizeof(T));
}

// Elements i to i + 3 of a float array, as lane_load (at any multiple of 4
// bytes).
typedef float rows4 __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ rows4 lane_load4(const float *base, int64_t at, int i) {
    typedef const __attribute__((address_space(1))) char *gchar_p;
    typedef const __attribute__((address_space(1))) rows4 *g_p;
    return *(g_p)((gchar_p)(base + at) + (uint32_t)i * 4u);
}

// A tile's pairs: the lane's column is j0 + jo, its rows start at i0 + io
// (i0 and j0 wavefront-uniform).
struct TilePos {
    int i0, j0, io, jo;
};

// The job record of the tiles, in constant memory: the paths that settle
// pairs one by one read its pointers when they need them (through an opaque
// copy of its address, so that the loads stay there), which leaves the scalar
// registers to the column loop.
typedef const __attribute__((address_space(4))) JobDev *cjob_p;
typedef const __attribute__((address_space(4))) PairArgs *cargs_p;

__device__ __forceinline__ cjob_p fresh(cjob_p p) {
    asm volatile("" : "+s"(p));
    return p;
}

// The rule's value of the pair at row offset i and column offset j.
template <bool M3>
__device__ __forceinline__ double rule_at(cjob_p job, const TilePos &t, int i, int j) {
    const cjob_p p = fresh(job);
    return rule_value<M3>(lane_load(p->ax64, t.i0, i), lane_load(p->ay64, t.i0, i), lane_load(p->az64, t.i0, i),
                          lane_load(p->bx64, t.j0, j), lane_load(p->by64, t.j0, j), lane_load(p->bz64, t.j0, j));
}

// Is row io + r of the tile past edge k against the lane's column?  FP32
// differences against the band, inside it the FP64 rule.
template <bool M3>
__device__ __forceinline__ bool past_edge(int q_exp2, cjob_p job, const Smem &s, int k, const TilePos &t, int r,
                                          Counters &cnt) {
    int i = t.io + r, j = t.jo;
    const cjob_p p = fresh(job);
    const float2 b = s.qband[k];
    const float q = diff_q(lane_load(p->ax32, t.i0, i), lane_load(p->ay32, t.i0, i), lane_load(p->az32, t.i0, i),
                           lane_load(p->bx32, t.j0, j), lane_load(p->by32, t.j0, j), lane_load(p->bz32, t.j0, j),
                           q_exp2);
    ++cnt.flag;
    if (q < b.x)
        return false;
    if (q >= b.y)
        return true;
    ++cnt.exact;
    return rule_at<M3>(job, t, i, j) <= s.D[k];
}

// The sixteen values of a lane as integers.
__device__ __forceinline__ void tile_bits(const floatx16 &acc, int32_t (&b)[16]) {
#pragma unroll
    for (int r = 0; r < 16; ++r)
        b[r] = (int32_t)__float_as_uint(acc[r]);
}

// Cell entries of the tiles (16 bits): the histogram row of the cell's slot,
// slot * rowstep, with kCellOpen set when an edge lies in the cell (the slot
// is then the lower one) and kCellMulti too when several do.  Rows are at
// least 16 bytes apart, so the flags are below them.
constexpr uint32_t kCellFlags = 15u;

__device__ __forceinline__ uint32_t cell_entry(float q, const Consts &k) {
    const int32_t c = med3_i32((int32_t)__float_as_uint(q) >> (int)k.shift, (int32_t)k.clo, (int32_t)k.chi);
    return *(const lds_u16 *)(uintptr_t)(((uint32_t)c << 1) + k.lutbias);
}

// What the tiles use of the launch's arguments.
struct TileArgs {
    int32_t nedges, q_exp2;
};

// Histogram row of one pair (row io, column jo) from FP32 differences and,
// where its cell or an edge's band leaves it open, the FP64 rule.
template <bool M3>
__device__ __forceinline__ uint32_t settle_row(const TileArgs &a, cjob_p job, const Smem &s, const Consts &k,
                                               const TilePos &t, Counters &cnt) {
    const cjob_p p = fresh(job);
    const float q = diff_q(lane_load(p->ax32, t.i0, t.io), lane_load(p->ay32, t.i0, t.io),
                           lane_load(p->az32, t.i0, t.io), lane_load(p->bx32, t.j0, t.jo),
                           lane_load(p->by32, t.j0, t.jo), lane_load(p->bz32, t.j0, t.jo), a.q_exp2);
    const uint32_t ent = cell_entry(q, k), row = ent & ~kCellFlags;
    if (!(ent & kCellOpen))
        return row;
    if (!(ent & kCellMulti)) {
        const float2 b = s.qband[row >> k.rowlog];
        if (q < b.x)
            return row;
        if (q >= b.y)
            return row + k.rowstep;
    }
    ++cnt.exact;
    return count_le(rule_at<M3>(job, t, t.io, t.jo), s.D, a.nedges) * k.rowstep;
}

// Bin one tile with a table lookup per pair, by squared distances q that lie
// within e of those of the FP32 copies (and within 2^-10 of them, for which
// the cells hold); the first w of the lane's rows count.  Pairs of cells that
// hold an edge compare q -+ e with its band; those inside it go to the
// discard row and are settled afterwards, from FP32 differences and by the
// FP64 rule.
template <bool M3>
__device__ __forceinline__ void tile_cells(const TileArgs &a, cjob_p job, const Smem &s, const Consts &k,
                                           const float (&q)[16], float e, const TilePos &t, uint32_t w,
                                           Counters &cnt) {
    uint32_t open = 0;      // bit r: pair r is not settled yet
    const uint32_t discard = (uint32_t)(a.nedges + 1) * k.rowstep;
    const bool part = __builtin_amdgcn_ballot_w64(w != 16u) != 0;
#pragma unroll
    for (int b = 0; b < 16; b += 4) {
        uint32_t ent[4];
#pragma unroll
        for (int r = 0; r < 4; ++r)
            ent[r] = cell_entry(q[b + r], k);
        if (__builtin_amdgcn_ballot_w64(((ent[0] | ent[1] | ent[2] | ent[3]) & kCellOpen) != 0) != 0) {
            // on every lane: a certain pair's row stays (an edge's band read
            // for it decides nothing)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const uint32_t row = ent[r] & ~kCellFlags;
                const float2 bd = s.qband[min(row >> k.rowlog, (uint32_t)(a.nedges - 1))];
                const bool one = (ent[r] & kCellFlags) == kCellOpen, edge = (ent[r] & kCellOpen) != 0;
                const uint32_t up = q[b + r] - e >= bd.y ? row + k.rowstep : q[b + r] + e < bd.x ? row : discard;
                ent[r] = edge ? one ? up : discard : row;
                open |= edge && ent[r] == discard ? 1u << (b + r) : 0u;
                cnt.flag += edge && (uint32_t)(b + r) < w ? 1u : 0u;
            }
        }
        if (part) {
#pragma unroll
            for (int r = 0; r < 4; ++r)
                ent[r] = (uint32_t)(b + r) < w ? ent[r] : discard;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
            lds_inc(ent[r] + k.lanebase);
        __builtin_amdgcn_sched_barrier(0);
    }
    open &= (1u << w) - 1u;
    if (__builtin_amdgcn_ballot_w64(open != 0) == 0)
        return;
    ++cnt.rare;
    while (open) {
        TilePos p = t;
        p.io += __builtin_ctz(open);
        open &= open - 1u;
        lds_inc(settle_row<M3>(a, job, s, k, p, cnt) + k.lanebase);
    }
}

// Squared distances of one tile from FP32 differences.  Four rows a load: with
// one, the 51 loads of a tile took a compute unit's address unit 816 cycles,
// 6 us a tile where every wavefront had one (DR of 1e4 x 1e4), and 12 to 20 %
// of all wavefront time from 1e4 to 1.5e5 points.  Where rows are missing,
// those past the last (offset ilast) read that one.
__device__ __forceinline__ void tile_diffs(const TileArgs &a, cjob_p job, const TilePos &t, int ilast,
                                           float (&q)[16]) {
    int io = t.io;
    asm volatile("" : "+v"(io));
    const cjob_p p = fresh(job);
    const float xj = lane_load(p->bx32, t.j0, t.jo), yj = lane_load(p->by32, t.j0, t.jo),
                zj = lane_load(p->bz32, t.j0, t.jo);
    if (__builtin_amdgcn_ballot_w64(io + 15 > ilast) == 0) {
#pragma unroll
        for (int b = 0; b < 16; b += 8) {
            rows4 x[2], y[2], z[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                x[h] = lane_load4(p->ax32, t.i0, io + b + 4 * h);
                y[h] = lane_load4(p->ay32, t.i0, io + b + 4 * h);
                z[h] = lane_load4(p->az32, t.i0, io + b + 4 * h);
            }
#pragma unroll
            for (int r = 0; r < 8; ++r)
                q[b + r] = diff_q(x[r >> 2][r & 3], y[r >> 2][r & 3], z[r >> 2][r & 3], xj, yj, zj, a.q_exp2);
            __builtin_amdgcn_sched_barrier(0);
        }
        return;
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int i = min(io + r, ilast);
        q[r] = diff_q(lane_load(p->ax32, t.i0, i), lane_load(p->ay32, t.i0, i), lane_load(p->az32, t.i0, i), xj, yj,
                      zj, a.q_exp2);
        if (r == 7)
            __builtin_amdgcn_sched_barrier(0);
    }
}

// Longest run of edges tile_count compares every pair with: an edge costs
// about 50 instructions a lane, a lookup tile as much as nine of them in LDS
// reads and atomics.
constexpr uint32_t kMaxSpan = 6;

// Slots of a lane's pairs from the cells of its smallest and largest q
// (within e): the lowest slot's histogram row and the number of edges above
// it.
__device__ __forceinline__ void tile_span(const float (&q)[16], float e, const Consts &k, uint32_t &row,
                                          uint32_t &span) {
    const float qmin = tree_reduce(q, [](float x, float y) { return fminf(x, y); });
    const float qmax = tree_reduce(q, [](float x, float y) { return fmaxf(x, y); });
    const uint32_t lo = cell_entry(qmin - e, k), hi = cell_entry(qmax + e, k);
    row = lo & ~kCellFlags;
    // a cell with several edges says nothing: too long a span
    span = ((hi - row) >> k.rowlog) + (hi & kCellOpen);
    span = (lo | hi) & kCellMulti ? ~0u : span;
}

// Bin one tile by comparing every pair with the lane's `span` edges above
// histogram row `row`: the pairs before an edge and not before the one below
// it go to the slot between them.  q lies within e of the squared distances
// of the FP32 copies; the first w of the lane's rows count.
template <bool M3>
__device__ __forceinline__ void tile_count(const TileArgs &a, cjob_p job, const Smem &s, const Consts &k,
                                           const float (&q)[16], float e, uint32_t row, uint32_t span,
                                           const TilePos &t, uint32_t w, Counters &cnt) {
    const uint32_t counted = 0xFFFF0000u >> w & 0xFFFFu;    // bit 15 - r: pair r counts
    uint32_t prev = 0, at = row + k.lanebase, ke = row >> k.rowlog, rare = 0;
#pragma unroll 1
    for (;; ++ke, at += k.rowstep, --span) {
        // span: edges left (counted down past 0 on lanes that are done)
        const bool on = (int32_t)span > 0;
        if (__builtin_amdgcn_ballot_w64(on) == 0)
            break;
        float2 b = s.qband[min(ke, (uint32_t)(a.nedges - 1))];
        asm volatile("" : "+v"(b.x), "+v"(b.y));            // read on every lane: no branch
        const float thr = b.y + e;
        const int32_t lim = on ? (int32_t)__float_as_uint(__fmaf_rn(-2.0f, e, b.x - b.y)) : INT32_MIN;
        uint32_t before = 0;
        int32_t near = INT32_MAX;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const uint32_t x = __float_as_uint(q[r] - thr);
            before = __builtin_amdgcn_alignbit(before, x, 31);
            near = min(near, (int32_t)x);
        }
        asm volatile("" : "+v"(before));
        if (__builtin_amdgcn_ballot_w64(near <= lim) != 0) {
            uint32_t und = 0;   // bit 15 - r: pair r is undecided
#pragma unroll
            for (int r = 0; r < 16; ++r)
                und = und * 2u + ((int32_t)__float_as_uint(q[r] - thr) <= lim ? 1u : 0u);
            und &= counted;
            rare = 1;
            while (und) {
                const int bit = __builtin_ctz(und);
                und &= und - 1u;
                const bool past = past_edge<M3>(a.q_exp2, job, s, (int)ke, t, 15 - bit, cnt);
                before = past ? before & ~(1u << bit) : before;
            }
        }
        // a lane past its last edge adds what is left to that edge's upper
        // slot, once
        const uint32_t n = on ? (uint32_t)__builtin_popcount(before & counted) : w;
        if ((int32_t)span >= 0)
            lds_add(at, n - prev);
        prev = n;
    }
    if (span == 0)
        lds_add(at, w - prev);
    cnt.rare += rare;
}

// q^ (less what c takes off) of one tile.
__device__ __forceinline__ floatx16 tile_q(const Frag &fa, const Frag &fb, const floatx16 &c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(fa.h, fb.h, c, 0, 0, 0);
}

// Row operands of G groups, four words each.
typedef uint32_t uintx32 __attribute__((ext_vector_type(32)));

__device__ __forceinline__ Frag rows_at(const uintx32 &fa, int g) {
    Frag f;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        f.d[i] = fa[4 * g + i];
    return f;
}

__device__ __forceinline__ void broadcast(floatx16 &c, float v) {
#pragma unroll
    for (int r = 0; r < 16; ++r)
        c[r] = v;
}

// bits = 2 bits + (any lane's bit set), on the scalar unit.
__device__ __forceinline__ void push_any(uint32_t &bits, uint64_t lanes) {
    asm("s_cmp_lg_u64 %1, 0\n\ts_addc_u32 %0, %0, %0" : "+s"(bits) : "s"(lanes) : "scc");
}

// Values of 64 columns, one per lane, dealt to the lanes of two tiles of 32
// columns (each column in lane and lane + 32): lo holds those of columns
// 0-31, hi those of columns 32-63.
__device__ __forceinline__ void deal(uint32_t v, uint32_t &lo, uint32_t &hi) {
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    lo = r[0];
    hi = r[1];
}

// The same for operands whose lower half takes v and whose upper half takes
// u of the same columns.
__device__ __forceinline__ void deal2(uint32_t v, uint32_t u, uint32_t &lo, uint32_t &hi) {
    const auto r = __builtin_amdgcn_permlane32_swap(v, u, false, false);
    lo = r[0];
    hi = r[1];
}

// Is e at most kTileFar of every counted q of the wavefront?
__device__ __forceinline__ bool far_enough(const float (&q)[16], float e, uint32_t w) {
    const float qmin = tree_reduce(q, [](float x, float y) { return fminf(x, y); });
    return __builtin_amdgcn_ballot_w64(!(qmin * kTileFar > e) && w) == 0;
}

// Columns [j, j + 64) of a catalog (x at b, y and z each `stride` elements
// further) into the wavefront's LDS buffer (x, y, z of 64 floats at byte
// address dst), straight from memory: the copy in flight takes no registers.
// Buffer loads, whose lane offset never changes and whose range makes columns
// from `end` on read as 0: with global loads each pass of 64 columns formed
// three 64-bit addresses a lane from three kept pointers.
__device__ __forceinline__ void stage_columns(const float *b, int64_t stride, int j, int end, int lane,
                                              uint32_t dst) {
    typedef __attribute__((address_space(3))) void *lds_p;
    const uint32_t bytes = 4u * (uint32_t)min(end - j, 64);
    asm volatile("" : "+v"(lane), "+s"(dst));       // (addresses formed here, not kept)
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const auto r = __builtin_amdgcn_make_buffer_rsrc((void *)(b + c * stride + j), 0, bytes, 0x00020000);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_p)(uintptr_t)(dst + 256u * c), 4, 4 * lane, 0, 0, 0);
    }
}

// nb and histogram row (~0 for a lane whose column does not exist) of the
// lane's column in the tile of columns h (0 or 32) on.
__device__ __forceinline__ void column_state(int h, float nb, uint32_t row, bool valid, float &nbh, uint32_t &rowh) {
    uint32_t n0, n1, r0, r1;
    deal(__float_as_uint(nb), n0, n1);
    deal(valid ? row : ~0u, r0, r1);
    nbh = __uint_as_float(h ? n1 : n0);
    rowh = h ? r1 : r0;
}

// The G tiles of 32 columns, x = q^ - (L + e) from the accumulator input: bit
// g is set when some lane's pairs of tile g are not all in the lane's slot (a
// pattern at or above `width`).  No branch between the tiles, and the matrix
// core works on the next tile while this one is reduced.
template <int G>
__device__ __forceinline__ uint32_t tile_screen(const uintx32 &fa, const Frag &fb, float base, uint32_t width) {
    floatx16 c;
    broadcast(c, base);
    uint32_t mask = 0;
    floatx16 acc = tile_q(rows_at(fa, G - 1), fb, c);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int g = G - 1; g >= 0; --g) {
        const floatx16 cur = acc;
        if (g > 0)
            acc = tile_q(rows_at(fa, g - 1), fb, c);
        __builtin_amdgcn_sched_barrier(0);
        int32_t x[16];
        tile_bits(cur, x);
        const uint32_t top = (uint32_t)tree_reduce(
            x, [](int32_t u, int32_t v) { return (int32_t)max((uint32_t)u, (uint32_t)v); });
        push_any(mask, __builtin_amdgcn_ballot_w64(top >= width));
        __builtin_amdgcn_sched_barrier(0);
    }
    return mask;
}

// One tile against edge k, x = q^ - (qhi_k + e): adds the lane's number of
// pairs before the edge to n_before.  room bounds |x| so that no other edge
// is reached, lim is the bit pattern of -((qhi_k - qlo_k) + 2e): x in
// [that, 0) leaves a pair undecided.  On signed bit patterns the decided x
// lie above lim (a negative float's pattern grows with its magnitude), so one
// signed minimum checks every pair.  False, with nothing counted, when some
// lane needs more than one edge or has more than three undecided pairs.
template <bool M3>
__device__ __forceinline__ bool tile_split(int q_exp2, cjob_p job, const Smem &s, const floatx16 &x, int k,
                                           float room, int32_t lim, const TilePos &t, uint32_t &n_before,
                                           Counters &cnt) {
    float ax[16];
    int32_t b[16];
    tile_bits(x, b);
#pragma unroll
    for (int r = 0; r < 16; ++r)
        ax[r] = fabsf(x[r]);
    const float far = tree_reduce(ax, [](float u, float v) { return fmaxf(u, v); });
    if (__builtin_amdgcn_ballot_w64(!(far < room)) != 0)
        return false;
    const int32_t near = tree_reduce(b, [](int32_t u, int32_t v) { return min(u, v); });
    uint32_t before = 0;    // bit 15 - r: pair r is before the edge
#pragma unroll
    for (int r = 0; r < 16; ++r)
        before = __builtin_amdgcn_alignbit(before, (uint32_t)b[r], 31);
    if (__builtin_amdgcn_ballot_w64(near <= lim) != 0) {
        uint32_t und = 0;   // bit 15 - r: pair r is undecided
#pragma unroll
        for (int r = 0; r < 16; ++r)
            und = und * 2u + (b[r] <= lim ? 1u : 0u);
        if (__builtin_amdgcn_ballot_w64(__builtin_popcount(und) > 3) != 0)
            return false;
        ++cnt.rare;
        while (und) {
            const int bit = __builtin_ctz(und);
            und &= und - 1u;
            const bool past = past_edge<M3>(q_exp2, job, s, k, t, 15 - bit, cnt);
            before = past ? before & ~(1u << bit) : before;
        }
    }
    n_before += (uint32_t)__builtin_popcount(before);
    return true;
}

// Low n bits, n clamped to [0, G].
template <int G>
__device__ __forceinline__ uint32_t low_bits(int n) {
    return (1u << min(max(n, 0), G)) - 1u;
}

// One wavefront: rows [ib, ie) (at most 32 G) against columns [j0, j1), with
// PRUNE those of the aligned blocks that `left` names (bit 0: j0's).
template <int G, bool M3, bool PRUNE>
__device__ void rows_tiles(cargs_p args, cjob_p job, const Smem &s, const Consts &k, int ib, int ie, int j0, int j1,
                           uint64_t left, int lane, Counters &cnt) {
    const int half = lane >> 5;
    const float S = args->q_scale, q_small = args->q_small;
    const TileArgs a{args->nedges, args->q_exp2};
    const bool auto_pairs = job->auto_pairs != 0;
    uintx32 fa;
    float cx, cy, cz, rho2 = 0.0f;
    {
        // matrix row m of a group is row 16 ((m >> 2) & 1) + 4 (m >> 3) + (m & 3)
        const int m = lane & 31, row = 16 * ((m >> 2) & 1) + 4 * (m >> 3) + (m & 3);
        float x[G], y[G], z[G], sx = 0.0f, sy = 0.0f, sz = 0.0f;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int i = min(32 * g + row, ie - 1 - ib);
            x[g] = lane_load(job->ax32, ib, i);
            y[g] = lane_load(job->ay32, ib, i);
            z[g] = lane_load(job->az32, ib, i);
            sx += x[g];
            sy += y[g];
            sz += z[g];
        }
        const float f = S / (float)(G * kWaveSize);
        cx = uniform_f(wave_sum_f(sx) * f);
        cy = uniform_f(wave_sum_f(sy) * f);
        cz = uniform_f(wave_sum_f(sz) * f);
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const float xs = __fmaf_rn(x[g], S, -cx), ys = __fmaf_rn(y[g], S, -cy), zs = __fmaf_rn(z[g], S, -cz);
            const float na = __fmaf_rn(zs, zs, __fmaf_rn(ys, ys, xs * xs));
            rho2 = fmaxf(rho2, na);
            const uint32_t v0 = split_f16(-2.0f * (half ? zs : xs), 1.0f);
            const uint32_t v1 = split_f16(half ? na * kNormScale : -2.0f * ys, half ? kNormLow : 1.0f);
            fa[4 * g] = v0;
            fa[4 * g + 1] = swap_f16(v0);
            fa[4 * g + 2] = v1;
            fa[4 * g + 3] = half ? 0u : swap_f16(v1);
        }
        rho2 = uniform_f(wave_max_f(rho2));
    }
    const float u = 5.9604644775390625e-08f;
    const float e_rows = uniform_f(u * (kTileErrA * rho2 + kTileErr0));
    const uint32_t b_const = pack_f16((_Float16)16384.0f, (_Float16)16.0f);
    const uint32_t overflow = (uint32_t)a.nedges << k.rowlog;
    // tiles whose rows all exist, and those with any
    const int nr = ie - ib;
    const uint32_t rows_ok = low_bits<G>(nr >> 5), rows_any = low_bits<G>((nr + 31) >> 5);
    uint32_t n_beyond = 0;
    // (registers of their own: else every pass reloads the eight that the job's
    // pointers were read into)
    const float *b;
    asm volatile("s_mov_b64 %0, %1" : "=s"(b) : "s"(job->bx32));
    uint32_t stride = (uint32_t)(job->by32 - job->bx32);
    asm volatile("" : "+s"(stride));
    // the next 64 columns are on their way into LDS while these are used
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t stage = s.stage_addr + wave * (uint32_t)kStageWaveBytes;
    typedef volatile __attribute__((address_space(3))) float *lfloat_p;
    const lfloat_p col = (lfloat_p)(uintptr_t)(stage + 4u * (uint32_t)lane);
    const int b0 = j0 >> 6;
    int j = j0, jn;
    if (PRUNE)
        j = max(j0, (b0 + __builtin_ctzll(left)) << 6);
    stage_columns(b, stride, j, j1, lane, stage);
    for (; j < j1; j = jn) {
        // this pass's columns end at jl (pruned launches: with their block),
        // the next one's start at jn
        const int jl = PRUNE ? min(j1, (j & ~63) + 64) : j1;
        jn = j + 64;
        if (PRUNE) {
            left &= left - 1u;
            jn = left ? (b0 + __builtin_ctzll(left)) << 6 : j1;
        }
        // each lane prepares one of 64 columns, then the values are dealt to
        // the two tiles of 32
        __builtin_amdgcn_s_waitcnt(0x0F70);     // vmcnt(0): the copy has landed
        float xn = col[0], yn = col[64], zn = col[128];
        asm volatile("" : "+v"(xn), "+v"(yn), "+v"(zn));
        const float xs = __fmaf_rn(xn, S, -cx), ys = __fmaf_rn(yn, S, -cy), zs = __fmaf_rn(zn, S, -cz);
        const float nb = __fmaf_rn(zs, zs, __fmaf_rn(ys, ys, xs * xs));
        Frag f;
        uint32_t f1[2], base, base1, width, width1;
        deal2(split_f16(xs, 1.0f), split_f16(zs, 1.0f), f.d[0], f1[0]);
        deal2(split_f16(ys, 1.0f), b_const, f.d[2], f1[1]);
        // the slot of the column's distance from the rows' mean: its row in
        // the histogram, lower end and width
        const uint32_t row = cell_entry(nb, k) & ~kCellFlags;
        const bool valid = j + lane < jl;
        {
            const float2 sl = s.slots[row >> k.rowlog];
            const float es = __fmaf_rn(8.0f * u, fabsf(sl.x), __fmaf_rn(u * kTileErrN, nb, e_rows));
            const uint32_t wd = __float_as_uint(fmaxf(__fmaf_rn(-2.0f, es, sl.y), 0.0f));
            deal(__float_as_uint(nb - (sl.x + es)), base, base1);
            deal(valid ? wd : ~0u, width, width1);
        }
        // the next copy starts here, when this one's columns and the tables
        // have been read (the compiler waits for copies in flight before any
        // LDS read) and the tiles of one pass are still to come
        asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(base), "+v"(width) : : "memory");
        if (jn < j1)
            stage_columns(b, stride, jn, j1, lane, stage);
        uint32_t n_in = 0;      // tiles in one slot: columns 0-31, columns 32-63 (<< 16)
#pragma unroll 1
        for (int h = 0; h < 64; h += 32) {
            f.d[1] = f.d[0];
            f.d[3] = f.d[2];    // (the rows' fourth word is 0 in the upper half)
            // tiles all of whose pairs count (for auto-pairs: every column
            // after every row), and those where some do
            uint32_t ok = rows_ok, any = rows_any;
            const int jh = j + h;
            if (auto_pairs) {
                ok &= low_bits<G>((jh - ib) >> 5);
                any &= low_bits<G>((min(jh + 31, jl - 1) - ib + 31) >> 5);
            }
            if (jh >= jl)
                any = ok = 0;
            uint32_t rest = any & ~ok;
            if (ok) {
                uint32_t todo = ok & tile_screen<G>(fa, f, __uint_as_float(base), width);
                n_in += (uint32_t)__builtin_popcount(ok & ~todo) << (h >> 1);
                if (todo) {
                    // the nearest edge of every column: its slot's upper one
                    // above the slot's middle, else the lower one
                    float nbh, eh;
                    uint32_t ke;
                    column_state(h, nb, row, valid, nbh, ke);
                    const bool vh = ke != ~0u;
                    ke = min(ke >> k.rowlog, (uint32_t)a.nedges);
                    eh = __fmaf_rn(u * kTileErrN, nbh, e_rows);
                    const float2 sl = s.slots[ke];
                    ke = nearest_edge(ke, nbh, sl.x, sl.y, (uint32_t)a.nedges);
                    const float4 ed = s.edges[ke];      // qhi, qhi - qlo, room below, above
                    eh = __fmaf_rn(8.0f * u, ed.x, eh);
                    const float room = vh ? fminf(ed.z, __fmaf_rn(-2.0f, eh, ed.w)) : __builtin_huge_valf();
                    const int32_t lim = vh ? (int32_t)__float_as_uint(__fmaf_rn(-2.0f, eh, -ed.y)) : INT32_MIN;
                    const float off = nbh - (ed.x + eh);
                    uint32_t n_before = 0, nd = 0;
                    while (todo) {
                        const int g = __builtin_ctz(todo);
                        todo &= todo - 1u;
                        const TilePos t{ib, j, 32 * g + 16 * half, min(h + (lane & 31), jl - 1 - j)};
                        floatx16 c;
                        broadcast(c, off);
                        if (tile_split<M3>(a.q_exp2, job, s, tile_q(rows_at(fa, g), f, c), (int)ke, room, lim, t,
                                           n_before, cnt))
                            ++nd;
                        else
                            rest |= 1u << g;
                    }
                    if (nd) {
                        if (vh) {
                            const uint32_t at = (ke << k.rowlog) + k.lanebase;
                            lds_add(at, n_before);
                            lds_add(at + k.rowstep, 16u * nd - n_before);
                        }
                        cnt.two_slot_steps += nd;
                    }
                }
            }
            while (rest) {
                const int g = __builtin_ctz(rest);
                rest &= rest - 1u;
                const TilePos t{ib, j, 32 * g + 16 * half, min(h + (lane & 31), jl - 1 - j)};
                const int jc = jh + (lane & 31), last = (auto_pairs ? min(ie, jc) : ie) - ib;
                const uint32_t w = jc < jl ? (uint32_t)min(max(last - t.io, 0), 16) : 0u;
                float nbh;
                uint32_t row_h;
                column_state(h, nb, row, valid, nbh, row_h);
                floatx16 c;
                broadcast(c, nbh);
                c = tile_q(rows_at(fa, g), f, c);
                float q[16];
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    q[r] = c[r];
                float eh = __fmaf_rn(u * kTileErrN, nbh, e_rows);
                // close pairs, where e is not small against q^, from FP32
                // differences
                uint32_t at, span;
                if (!far_enough(q, eh, w)) {
                    tile_diffs(a, job, t, ie - 1 - ib, q);
                    eh = 0.0f;
                }
                tile_span(q, eh, k, at, span);
                span = w ? span : 0u;
                if (__builtin_amdgcn_ballot_w64(span > kMaxSpan) == 0)
                    tile_count<M3>(a, job, s, k, q, eh, at, span, t, w, cnt);
                else
                    tile_cells<M3>(a, job, s, k, q, eh, t, w, cnt);
            }
            f.d[0] = f1[0];
            f.d[2] = f1[1];
            base = base1;
            width = width1;
        }
        if (n_in) {
            const uint32_t both = (n_in & 0xFFFFu) + (n_in >> 16);
            if (j + 64 <= jl && __builtin_amdgcn_ballot_w64(row != overflow) == 0) {
                n_beyond += both;
            } else {
                lds_add(row + k.lanebase, valid ? 32u * (half ? n_in >> 16 : n_in & 0xFFFFu) : 0u);
                cnt.one_slot_steps += both;
            }
        }
        // work statistic: steps whose columns lie close to the rows
        if (__builtin_amdgcn_ballot_w64(nb < q_small) != 0)
            cnt.chord_steps += 2 * G;
    }
    cnt.beyond_steps += n_beyond;
    cnt.beyond += n_beyond * 16u;
}

// The next work item, or n_items when none is left.  Items past the first
// n_waves are dealt to kQueues counters in turn, each on a line of its own: an
// atomic add on one address takes the device 11 ns whoever asks, and 4096
// wavefronts asking one counter for their first item waited 22 us on average
// (45 at most), then again to learn that none was left: DD+DR+RR of 1e4 x 1e4
// 0.495 -> 0.34 ms, pruned 5e5 x 1e6 49.6 -> 48.2 ms.  Also measured, with one
// counter: several items at a time, which slowed every large launch (a 3-D
// box of 5e5 x 1e6 55.2 -> 59.7 ms, 64 regions 6.4 -> 7.5).  A wavefront whose
// counter is exhausted goes to the next one that has items left; every
// counter fails it at most once, so every wavefront leaves.
__device__ __forceinline__ uint32_t claim_item(unsigned int *queues, uint32_t n_waves, uint32_t n_items, uint32_t &q,
                                               int lane) {
    const uint32_t rest = n_items - min(n_waves, n_items);
    uint32_t open = (1u << kQueues) - 1u;
    if (rest == 0)
        return n_items;
    // where most wavefronts have no second item, they look before they ask
    bool look = rest < n_waves;
    while (open) {
        if (look) {
            const uint32_t l = (uint32_t)lane & (kQueues - 1);
            const uint32_t used =
                __hip_atomic_load(queues + l * kQueueStride, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            open &= (uint32_t)__builtin_amdgcn_ballot_w64(used < (rest + kQueues - 1u - l) / kQueues);
            if (!open)
                break;
            const uint32_t from = open & ~((1u << q) - 1u);     // this one or the next with items left
            q = (uint32_t)__builtin_ctz(from ? from : open);
        }
        uint32_t n = 0;
        if (lane == 0)
            n = atomicAdd(queues + q * kQueueStride, 1u);
        n = __builtin_amdgcn_readfirstlane(n);
        if (n < (rest + kQueues - 1u - q) / kQueues)
            return n_waves + n * kQueues + q;
        open &= ~(1u << q);
        look = true;
    }
    return n_items;
}

// PREC: 2 FP32 tiles, 1 FP64 vector; 3-D distances: 3 FP32 tiles, 4 FP64
// vector.  P: rows per lane (a wavefront covers P * 64 rows of a unit, for
// tiles 2 P groups of 32).
template <int PREC, bool LUT8, int P, bool PRUNE>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(waves_per_eu_of(PREC)))) void pairs_kernel(
    PairArgs a) {
    constexpr int kRowsPerWave = P * kWaveSize;
    extern __shared__ __align__(16) unsigned char smem[];
    const Smem s = carve<PREC == 2 || PREC == 3>(smem, a);
    const int tid = threadIdx.x;
    const int lane = tid & (kWaveSize - 1);
    const int wave = tid >> 6;

    const int hist_words = kWaves * (a.nslots + 1) * a.hist_copies;
    // 16 bytes a lane (hist_words is a multiple of 16, the device table is
    // padded to 16 bytes and so is its place in LDS): with one element a lane
    // this copy took longer than the pairs of a small launch
    for (int w = tid; w < hist_words / 4; w += kBlock)
        reinterpret_cast<uint4 *>(s.hist)[w] = make_uint4(0, 0, 0, 0);
    const int lut_words = (a.lut_cells * (LUT8 ? 1 : 2) + 15) / 16;
    for (int w = tid; w < lut_words; w += kBlock)
        reinterpret_cast<uint4 *>(s.lut)[w] = reinterpret_cast<const uint4 *>(a.lut)[w];
    for (int e = tid; e < a.nedges; e += kBlock) {
        s.D[e] = a.D[e];
        if (PREC == 2 || PREC == 3) {
            s.qband[e] = make_float2(a.qlo[e], a.qhi[e]);
            s.edges[e] = a.tile_edges[e];
        } else {
            s.E[e] = a.E[e];
        }
    }
    if (PREC == 2 || PREC == 3)
        for (int e = tid; e < a.nslots; e += kBlock)
            s.slots[e] = a.tile_slots[e];
    __syncthreads();

    Consts k;
    k.shift = (uint32_t)a.lut_shift;
    k.clo = to_vgpr((uint32_t)a.lut_lo);
    k.chi = to_vgpr((uint32_t)a.lut_hi);
    k.lutbias = s.lut_addr - (uint32_t)a.lut_lo * (LUT8 ? 1u : 2u);
    k.rowstep = (uint32_t)a.hist_copies * 4u;
    k.rowlog = 31u - (uint32_t)__builtin_clz(k.rowstep);
    k.flag = to_vgpr(Code<LUT8>::flag);
    k.beyond = to_vgpr(a.beyond_key);
    k.by_dot = a.beyond_dot != 0;
    k.lanebase = s.hist_addr +
                 (uint32_t)((wave * (a.nslots + 1) * a.hist_copies + (lane & (a.hist_copies - 1))) * 4);
    Counters cnt;

    uint32_t n_skip = 0;
    // Counts not flushed yet: where they go (the histogram and up to two
    // regions of the last items) and how many pairs they hold.  A wavefront
    // keeps them over its items until they go elsewhere or 2^31 pairs are
    // near (one LDS count holds less than 2^32): flushing 42 slots with
    // global atomics after every item cost about 12 ns of the device an item.
    unsigned long long *to = nullptr, *to_a = nullptr, *to_b = nullptr;
    uint32_t held = 0;
    const int copy = (int)((blockIdx.x * kWaves + (uint32_t)__builtin_amdgcn_readfirstlane(wave)) & (kGlobalCopies - 1));
    auto flush = [&]() {
        // pairs counted beyond the last edge go to this lane's copy of the
        // overflow slot; then the wave's own LDS region is flushed (no block
        // barrier needed)
        if (cnt.beyond) {
            lds_add(__umul24((uint32_t)(a.nslots - 1), k.rowstep) + k.lanebase, cnt.beyond);
            cnt.beyond = 0;
        }
        flush_wave(a, s, to, to_a, to_b, wave, lane, copy);
        held = 0;
    };
    // Each wavefront's first item is the one with its number, the others come
    // from the queues (claim_item), so the items in flight are always a window
    // of nearly consecutive units that share their column range (the plan
    // orders units column chunk first) and the column data stays in L2.
    const uint32_t n_items = (uint32_t)a.n_units * kWaves, n_waves = gridDim.x * kWaves;
    uint32_t queue = blockIdx.x & (kQueues - 1);
    int32_t unlooked = 1 << 21;     // pairs up to the next look (a cancellable launch holds one job)
    bool gone = false;
    for (uint32_t next = blockIdx.x * kWaves + (uint32_t)__builtin_amdgcn_readfirstlane(wave); next < n_items;
         next = claim_item(a.queue, n_waves, n_items, queue, lane)) {
        const int u = (int)(next / kWaves);
        const int part = (int)(next % kWaves);
        Unit un;
        if (a.units) {
            un = load_uniform(a.units + u);
        } else {
            un.job = 0;
            un.reg_a = un.reg_b = -1;
            if (!grid_unit(a.grid, (uint32_t)u, &un.i0, &un.i1, &un.j0, &un.j1))
                continue;
        }
        const cargs_p args = (cargs_p)__builtin_amdgcn_kernarg_segment_ptr();
        const cjob_p job = a.jobs ? (cjob_p)(a.jobs + un.job) : &args->job0;
        const JobDev jb = a.jobs ? load_uniform(a.jobs + un.job) : a.job0;
        const int ib = un.i0 + part * kRowsPerWave;
        // (auto-pairs: columns up to the first row count nothing)
        const int jb0 = jb.auto_pairs ? max(un.j0, ib + 1) : un.j0;
        if (ib < un.i1 && jb0 < un.j1) {
            const int ie = min(un.i1, ib + kRowsPerWave);
            const uint64_t pairs = (uint64_t)(ie - ib) * (uint64_t)(un.j1 - un.j0);
            // a cancelled job skips its remaining units; the flag lives in
            // host memory, which wavefronts read one after the other, 90 ns
            // each, so a wavefront looks at it every 2^21 pairs (about 0.6 ms
            // of its work), and in a short launch never: at every item, twelve
            // jobs of up to 3e10 pairs took 60 instead of 38 ms; with a look
            // at its first item too, a submitted DR of 637 x 55000 took 293
            // us, now 57, one of 1000 x 100000 567, now 116 (as tpcf_count)
            if (jb.cancel) {
                unlooked -= (int32_t)min(pairs, (uint64_t)1 << 21);
                if (unlooked <= 0) {
                    unlooked = 1 << 21;
                    gone = __builtin_amdgcn_readfirstlane(
                               __hip_atomic_load(jb.cancel, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM)) != 0;
                }
                if (gone) {
                    ++n_skip;
                    continue;
                }
            }
            unsigned long long *r0 = nullptr, *r1 = nullptr;
            if (jb.touch) {
                const size_t per_region = (size_t)kGlobalCopies * a.nslots;
                if (un.reg_a >= 0)
                    r0 = jb.touch + (size_t)un.reg_a * per_region;
                if (un.reg_b >= 0 && un.reg_b != un.reg_a)
                    r1 = jb.touch + (size_t)un.reg_b * per_region;
            }
            // (an item is at most 2^30 pairs, see make_grid)
            if (held && (to != jb.hist || to_a != r0 || to_b != r1 || held + pairs >= 0x80000000ull))
                flush();
            to = jb.hist;
            to_a = r0;
            to_b = r1;
            held = (uint32_t)min((uint64_t)held + pairs, (uint64_t)0xFFFFFFFFu);
            // columns [jb0, jm) need a test per pair: all of them when the
            // rows do not fill the wavefront, for auto-pairs those up to the
            // last row
            const int jm = ie - ib < kRowsPerWave ? un.j1 : jb.auto_pairs ? min(max(ie, jb0), un.j1) : jb0;
            if (PREC == 2 || PREC == 3) {
                constexpr bool M3 = PREC == 3;
                if (!PRUNE) {
                    rows_tiles<2 * P, M3, false>(args, job, s, k, ib, ie, jb0, un.j1, 0, lane, cnt);
                } else {
                    // aligned blocks past the masked columns, when every row
                    // exists and the catalog has caps
                    const bool caps = ie - ib == kRowsPerWave && jb.bcaps;
                    for (int jr = jb0, je; jr < un.j1; jr = je) {
                        je = part_end(jr, un.j1, kPruneCols - (jr & 63));
                        uint64_t left;
                        if (caps) {
                            double x[P], y[P], z[P];
#pragma unroll
                            for (int p = 0; p < P; ++p) {
                                x[p] = lane_load(job->ax32, ib, kWaveSize * p + lane);
                                y[p] = lane_load(job->ay32, ib, kWaveSize * p + lane);
                                z[p] = lane_load(job->az32, ib, kWaveSize * p + lane);
                            }
                            left = prune_blocks<M3>(block_cap<M3, P>(x, y, z), jb.bcaps, s, a, k, jr, je, jm,
                                                    kRowsPerWave * 64, lane, cnt);
                        } else {
                            left = blocks_met(jr, je);
                        }
                        if (left)
                            rows_tiles<2 * P, M3, true>(args, job, s, k, ib, ie, jr, je, left, lane, cnt);
                    }
                }
            } else {
                constexpr bool M3 = PREC == 4;
                if (jb0 < jm)
                    rows_fp64<LUT8, true, P, PRUNE, M3>(a, jb, s, k, ib, ie, jb0, jm, lane, cnt);
                if (jm < un.j1)
                    rows_fp64<LUT8, false, P, PRUNE, M3>(a, jb, s, k, ib, ie, jm, un.j1, lane, cnt);
            }
        }
    }
    if (held)
        flush();
    // work statistics: one lane per word, into one of kStatCopies copies
    // (thousands of wavefronts adding to one line would wait for each other
    // longer than a small launch runs)
    const uint32_t f = wave_sum(cnt.flag);
    const uint32_t x = wave_sum(cnt.exact);
    unsigned long long v = 0;
    switch (lane) {
    case 0: v = cnt.two_slot_steps; break;
    case 1: v = f; break;
    case 2: v = x; break;
    case 3: v = n_skip; break;
    case 4: v = cnt.rare; break;
    case 5: v = cnt.beyond_steps; break;
    case 6: v = cnt.one_slot_steps; break;
    case 7: v = (unsigned long long)cnt.pruned_blocks * (unsigned long long)(kRowsPerWave * 64); break;
    case 8: v = cnt.chord_steps; break;
    }
    if (v)
        atomicAdd(&a.stats[(size_t)(copy & (kStatCopies - 1)) * kStatStride + lane], v);
}

__global__ void zero_u64_kernel(unsigned long long *p, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride)
        p[i] = 0ull;
}

// One block per job: sum its kGlobalCopies histogram copies.  CLEAR (one job):
// also leave them, and the `queue` words after them, zero for the next launch.
template <bool CLEAR>
__global__ void reduce_copies_kernel(unsigned long long *copies, int32_t nslots, unsigned long long *out,
                                     int32_t queue) {
    unsigned long long *c = copies + (size_t)blockIdx.x * kGlobalCopies * nslots;
    for (int s = threadIdx.x; s < nslots; s += blockDim.x) {
        unsigned long long acc = 0;
#pragma unroll 16
        for (int g = 0; g < kGlobalCopies; ++g)
            acc += c[(size_t)g * nslots + s];
        out[(size_t)blockIdx.x * nslots + s] = acc;
        if (CLEAR)
#pragma unroll 16
            for (int g = 0; g < kGlobalCopies; ++g)
                c[(size_t)g * nslots + s] = 0;
    }
    if (CLEAR)
        for (int i = threadIdx.x; i < queue; i += blockDim.x)
            copies[(size_t)kGlobalCopies * nslots + i] = 0;
}

// FP32 copies (round to nearest) of an FP64 SoA block of 3n values, and the
// largest |x^2 + y^2 + z^2 - 1| (FP64, unfused), +inf if a value is not finite.
// With `given` (caller-owned FP32 copies) nothing is written: every given
// value is compared with the rounded FP64 one and *mismatch is set if one
// differs.
__global__ void to_float_kernel(const double *xyz, int64_t n, float *out, const float *given,
                                unsigned long long *maxdev, unsigned long long *mismatch) {
    __shared__ double red[256];
    double m = 0.0;
    bool differs = false;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        double x = xyz[i], y = xyz[n + i], z = xyz[2 * n + i];
        if (given) {
            differs = differs || given[i] != (float)x || given[n + i] != (float)y || given[2 * n + i] != (float)z;
        } else {
            out[i] = (float)x;
            out[n + i] = (float)y;
            out[2 * n + i] = (float)z;
        }
        double t = x * x;
        double u = y * y;
        double v = z * z;
        double r = (t + u) + v;
        double dev = fabs(r - 1.0);
        if (!isfinite(x) || !isfinite(y) || !isfinite(z) || !(dev == dev))
            dev = __builtin_huge_val();
        m = dev > m ? dev : m;
    }
    if (differs)
        atomicOr(mismatch, 1ull);
    red[threadIdx.x] = m;
    __syncthreads();
    for (int off = blockDim.x / 2; off > 0; off >>= 1) {
        if ((int)threadIdx.x < off)
            red[threadIdx.x] = red[threadIdx.x] > red[threadIdx.x + off] ? red[threadIdx.x] : red[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0)
        atomicMax(maxdev, (unsigned long long)__double_as_longlong(red[0]));
}

// Bounding cap of every aligned group of 64 stored points: one wavefront per
// group (4 doubles: unit centre, angular radius).
__global__ __launch_bounds__(256) void caps64_kernel(const double *xyz, int64_t n, double *caps,
                                                     int64_t groups, int metric) {
    const int lane = threadIdx.x & (kWaveSize - 1);
    const int wave = threadIdx.x >> 6;
    for (int64_t g = (int64_t)blockIdx.x * kWaves + wave; g < groups; g += (int64_t)gridDim.x * kWaves) {
        // lanes past the catalog repeat the group's first point
        const int64_t p = g * 64 + lane < n ? g * 64 + lane : g * 64;
        const double x[1] = {xyz[p]}, y[1] = {xyz[n + p]}, z[1] = {xyz[2 * n + p]};
        const Cap c = metric ? ball_of<1>(x, y, z) : cap_of<1>(x, y, z);
        if (lane == 0) {
            caps[4 * g] = c.x;
            caps[4 * g + 1] = c.y;
            caps[4 * g + 2] = c.z;
            caps[4 * g + 3] = c.rho;
        }
    }
}

int grid_for(int n_units, int lds, int blocks_per_cu) {
    static int cus = 0, lds_per_cu = 0;
    if (!cus) {
        int dev = 0;
        (void)hipGetDevice(&dev);
        hipDeviceProp_t prop;
        if (hipGetDeviceProperties(&prop, dev) == hipSuccess) {
            cus = prop.multiProcessorCount;
            lds_per_cu = (int)prop.maxSharedMemoryPerMultiProcessor;
        }
        if (cus <= 0)
            cus = 256;
        if (lds_per_cu <= 0)
            lds_per_cu = 160 * 1024;
    }
    int per_cu = lds > 0 ? lds_per_cu / lds : 8;
    if (per_cu < 1)
        per_cu = 1;
    if (per_cu > 8)
        per_cu = 8;
    // the resident blocks by default (the work queue balances them);
    // blocks_per_cu > 0 overrides
    long long g = blocks_per_cu > 0 ? (long long)cus * blocks_per_cu : (long long)cus * per_cu;
    if (g > n_units)
        g = n_units;
    if (g < 1)
        g = 1;
    return (int)g;
}

template <int PR, bool B8, bool PRUNE>
void launch_pairs(int P, int grid, int lds, hipStream_t st, const PairArgs &a) {
    if constexpr ((PR == 2 || PR == 3) && !PRUNE) {
        if (P == 1) {
            hipLaunchKernelGGL((pairs_kernel<PR, B8, 1, PRUNE>), dim3(grid), dim3(kBlock), lds, st, a);
            return;
        }
    }
    if (P == 2)
        hipLaunchKernelGGL((pairs_kernel<PR, B8, 2, PRUNE>), dim3(grid), dim3(kBlock), lds, st, a);
    else
        hipLaunchKernelGGL((pairs_kernel<PR, B8, 4, PRUNE>), dim3(grid), dim3(kBlock), lds, st, a);
}


}  // namespace

extern "C" int tpcf_launch_pairs(const PairArgs *args, int precision, void *stream) {
    if (args->n_units <= 0)
        return 0;
    const int lds = lds_bytes(args->nslots, args->hist_copies, args->lut_cells, args->lut_entry_bytes, args->nedges) +
                    (args->tile_slots ? tile_lds_bytes(args->nslots) : 0);
    const int grid = grid_for(args->n_units, lds, args->blocks_per_cu);
    hipStream_t st = (hipStream_t)stream;
    const bool b8 = args->lut_entry_bytes == 1;
    const int P = args->rows_per_lane;
    if (P != 2 && P != 4 && !(P == 1 && precision == 0 && !args->prune))
        return (int)hipErrorInvalidValue;
    const bool prune = args->prune != 0;
    if (precision != 0 && precision != 1)
        return (int)hipErrorInvalidValue;
    if (args->metric == 1) {
        if (precision == 0)
            prune ? launch_pairs<3, false, true>(P, grid, lds, st, *args) : launch_pairs<3, false, false>(P, grid, lds, st, *args);
        else if (prune)
            b8 ? launch_pairs<4, true, true>(P, grid, lds, st, *args) : launch_pairs<4, false, true>(P, grid, lds, st, *args);
        else
            b8 ? launch_pairs<4, true, false>(P, grid, lds, st, *args) : launch_pairs<4, false, false>(P, grid, lds, st, *args);
    } else {
        if (precision == 0)
            prune ? launch_pairs<2, false, true>(P, grid, lds, st, *args) : launch_pairs<2, false, false>(P, grid, lds, st, *args);
        else if (prune)
            b8 ? launch_pairs<1, true, true>(P, grid, lds, st, *args) : launch_pairs<1, false, true>(P, grid, lds, st, *args);
        else
            b8 ? launch_pairs<1, true, false>(P, grid, lds, st, *args) : launch_pairs<1, false, false>(P, grid, lds, st, *args);
    }
    return (int)hipGetLastError();
}

extern "C" int tpcf_launch_caps64(const double *xyz64, int64_t n, double *caps, int metric, void *stream) {
    const int64_t groups = (n + 63) / 64;
    if (groups <= 0)
        return 0;
    int64_t blocks = (groups + kWaves - 1) / kWaves;
    if (blocks > 4096)
        blocks = 4096;
    hipLaunchKernelGGL(caps64_kernel, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream, xyz64, n,
                       caps, groups, metric);
    return (int)hipGetLastError();
}

extern "C" int tpcf_launch_zero_u64(unsigned long long *p, int64_t n, void *stream) {
    if (n <= 0)
        return 0;
    int64_t blocks = (n + 255) / 256;
    if (blocks > 1024)
        blocks = 1024;
    hipLaunchKernelGGL(zero_u64_kernel, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream, p, n);
    return (int)hipGetLastError();
}

extern "C" int tpcf_launch_reduce_copies(unsigned long long *copies, int32_t nslots, int32_t njobs,
                                         unsigned long long *out, void *stream) {
    if (njobs <= 0)
        return 0;
    hipLaunchKernelGGL(reduce_copies_kernel<false>, dim3((unsigned)njobs), dim3(256), 0, (hipStream_t)stream,
                       copies, nslots, out, 0);
    return (int)hipGetLastError();
}

extern "C" int tpcf_launch_reduce_clear(unsigned long long *copies, int32_t nslots, int32_t queue_words,
                                        unsigned long long *out, void *stream) {
    hipLaunchKernelGGL(reduce_copies_kernel<true>, dim3(1), dim3(256), 0, (hipStream_t)stream, copies, nslots, out,
                       queue_words);
    return (int)hipGetLastError();
}

extern "C" int tpcf_launch_to_float(const double *xyz64, int64_t n, float *xyz32, const float *given32,
                                    unsigned long long *check_out, void *stream) {
    // check_out: two device words zeroed by the caller, [0] the largest norm
    // deviation (a double's bits), [1] non-zero if a given FP32 copy differs
    if (n <= 0)
        return 0;
    int64_t blocks = (n + 255) / 256;
    if (blocks > 2048)
        blocks = 2048;
    hipLaunchKernelGGL(to_float_kernel, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream,
                       xyz64, n, xyz32, given32, check_out, check_out + 1);
    return (int)hipGetLastError();
}

// ---------------------------------------------------------------------------
// Work area of the entry point that allocates nothing (tpcf_count_noalloc):
// a fixed array in device memory, one per device the library runs on, held
// until the process ends.  Host code never uses the array's name as an
// address (on the host it is only a stand-in for the symbol): the device
// address comes from hipGetSymbolAddress, looked up once per device with
// that device current, and kernels receive that pointer as an argument.
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {
constexpr int kMaxScratchDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxScratchDevices] = {};
}  // namespace

extern "C" int tpcf_scratch_init(int device) {
    if (device < 0 || device >= kMaxScratchDevices)
        return (int)hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (g_scratch_ptr[device])
        return 0;
    int cur = -1;
    hipError_t e = hipGetDevice(&cur);
    if (e != hipSuccess)
        return (int)e;
    if (cur != device)
        return (int)hipErrorInvalidDevice;      // the caller makes the device current first
    void *ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess)
        return (int)e;
    if (!ptr)
        return (int)hipErrorInvalidSymbol;
    g_scratch_ptr[device] = ptr;
    return 0;
}

extern "C" void *tpcf_scratch_ptr(int device) {
    if (device < 0 || device >= kMaxScratchDevices)
        return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    return g_scratch_ptr[device];
}
