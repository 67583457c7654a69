// HIP kernels of the reconstruction path for gfx950 and their launchers.
//
//   k_trace        ordered emission list of each proton's path (debug/parity)
//   k_forward      y = A x, ||a_i||^2   (one lane per proton, gathers)
//   k_backproject  g += A^T r           (one lane per proton, LDS lines, atomics)
//   k_drop_bin     DROP block, a wave per row: records -> a_i.x, ||a_i||^2 ->
//                  rho_i, chords into slab bins (FP32)
//   k_slab_commit  x_j += acc_j / s_j slab by slab from the bins
//   k_drop_block   DROP block, a wave per row, one atomic per piece (separate
//                  schedule); k_drop_fused: with the commit of the block before
//   k_drop_rows    the same with one lane per row
//   k_rows_bin     DROP block over stored rows: entries for k_slab_commit
//   k_drop_rows_fused  the same with atomics, and the commit of the block before
//   k_drop_commit  x_j += acc_j / s_j, reset
//   k_tv           smoothed total variation value and gradient
#include <hip/hip_ext.h>
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <climits>
#include <cstdint>
#include <cstring>
#include <mutex>
#include <type_traits>
#include <vector>

#include "pct_internal.h"
#include "pct_path.hpp"
#include "pct_lane_walk.hpp"
#include "pct_walk.hpp"

namespace pct {

__device__ __forceinline__ void raise_status(unsigned *status, unsigned bit)
{
    atomicOr(status, bit);
}

// Block-boundary gate of a cancellable DROP call (workspace header words).
// Every per-block kernel returns at once while the gate is closed; the last
// workgroup of each commit launch counts the block step and, when the host
// has requested a stop, closes the gate for the launches after it.  The
// gate word changes only there, after every workgroup of that launch has
// read it, so all workgroups of a launch take the same decision.
struct GateDev {
    int *halt;          // nullptr: the call is not cancellable
    unsigned *wg_done;  // workgroups of the running commit launch that ended
    const int *cancel;  // the host's request
    long long *done;    // block steps applied by the call
    unsigned *status;
};

__device__ __forceinline__ bool gate_closed(const int *halt) { return halt && *halt != 0; }

__device__ __forceinline__ void gate_commit_end(const GateDev &gt)
{
    if (!gt.halt) return;
    // every wave of the workgroup has read the gate (a load consumed by the
    // entry branch) before the workgroup is counted
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned k = atomicAdd(gt.wg_done, 1u);
        if (k == gridDim.x - 1) {
            *gt.wg_done = 0u;
            *gt.done += 1;
            if (__hip_atomic_load(gt.cancel, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) != 0) {
                *gt.halt = 1;
                atomicOr(gt.status, PCT_DEV_CANCELLED);
            }
        }
    }
}

// Start of a cancellable call: gate open, no block step applied.
__global__ void k_gate_begin(GateDev gt)
{
    if (threadIdx.x == 0) {
        *gt.halt = 0;
        *gt.wg_done = 0u;
        *gt.done = 0;
    }
}

// The whole path of one row, piece by piece, into sink.piece; false if the path
// does not move on along the row's dominant axis in every segment.
template <bool HULL, class Sink>
__device__ __forceinline__ bool walk_row(const Rec &r, const PathSrc &src, const GridDev &g, Sink &sink)
{
    const RowPath<HULL> path(src, g, r);
    LaneWalk<HULL> walk(path, g, r);
    walk.run(0, path.K, sink);
    walk.finish(sink);
    return walk.onward;
}

// ---------------------------------------------------------------------------
// trace
// ---------------------------------------------------------------------------
struct TraceSink {
    int32_t *vox;
    double *chord;
    int32_t cap, n;
    __device__ __forceinline__ void piece(int j, int, int, int, double c)
    {
        if (n < cap) {
            vox[n] = j;
            chord[n] = c;
        }
        ++n;
    }
};

template <bool HULL>
__global__ void __launch_bounds__(kWG) k_trace(ProtonsDev p, int64_t first, int64_t count, int32_t max_nnz,
                                               int32_t *vox, double *chord, int32_t *nnz,
                                               const PathSrc src,  GridDev g, unsigned *status)
{
    int64_t q = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (q >= count) return;
    Rec r = load_rec(p, first + q);
    TraceSink ts{vox + q * max_nnz, chord + q * max_nnz, max_nnz, 0};
    if (rec_finite(r)) {
        walk_row<HULL>(r, src, g, ts);
    } else {
        raise_status(status, PCT_DEV_NONFINITE);
    }
    nnz[q] = ts.n;
    if (ts.n > max_nnz) raise_status(status, PCT_DEV_ROW_OVERFLOW);
}

// ---------------------------------------------------------------------------
// forward projection
// ---------------------------------------------------------------------------
// Value of the iterate at voxel j seen by a block.
template <typename T>
struct PlainX {
    const T *__restrict__ x;
    __device__ __forceinline__ double operator()(int j) const { return double(x[j]); }
};

// The value read for a piece is used when the next piece comes, so the reads
// stay in flight behind the walk.
template <typename T, bool NORM, int CHORD = PCT_CHORD_F64>
struct DotSink {
    const T *__restrict__ x;
    Reentry *re;
    T pending = T(0);
    double c0 = 0.0, dot = 0.0, n2 = 0.0;
    __device__ __forceinline__ void piece(int j, int ix, int iy, int iz, double c)
    {
        c = round_chord<CHORD>(c);
        dot = fma(c0, double(pending), dot);
        pending = x[j];
        c0 = c;
        if constexpr (NORM) {
            bool first;
            const double before = re->visit(j, ix, iy, iz, c, first);
            n2 = fma(c, 2.0 * before + c, n2);
        }
    }
    __device__ __forceinline__ double sum() const { return fma(c0, double(pending), dot); }
};

// One lane per row: bound by FP64 instructions (about 80 a segment and 25 a
// crossing, 4 waves a SIMD, 3 with norms).  2e6 rows of 220 segments on the 256 x
// 256 x 64 grid: 2.6 ms, 3.65 with norms (5.8 for either with a walk from plane
// to plane of each segment's clipped part and a register window of pieces).
template <typename T, bool HULL, bool NORM>
__global__ void __launch_bounds__(kWG) k_forward(ProtonsDev p, int64_t first, int64_t n, const T *__restrict__ x,
                                                 T *y, T *nrm2, const PathSrc src, GridDev g, unsigned *status)
{
    int64_t i = first + int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    Rec r = load_rec(p, i);
    __shared__ std::conditional_t<NORM, Reentry::Lds, int> lds;
    Reentry re(reinterpret_cast<Reentry::Lds &>(lds), r);
    DotSink<T, NORM> s{x, &re};
    if (rec_finite(r)) {
        const bool onward = walk_row<HULL>(r, src, g, s);
        if (!onward || (NORM && re.unsafe)) raise_status(status, PCT_DEV_REENTRY);
    } else {
        raise_status(status, PCT_DEV_NONFINITE);
    }
    y[i] = T(s.sum());
    if constexpr (NORM) nrm2[i] = T(s.n2);
}

// ---------------------------------------------------------------------------
// back projection
// ---------------------------------------------------------------------------
// Back projection g += A^T r, one lane per proton.  HBM atomics bound it: about
// 2.3e10 lanes a second, wherever they point, unless neighbouring lanes name
// neighbouring voxels.  The 256 rows of a workgroup are consecutive in the scan,
// and an angle-sorted scan's consecutive rows cross nearly the same voxels, so
// the workgroup sums its pieces in an LDS table.  Its key is a line of eight
// consecutive voxels (open addressing, a few probes): the table then reaches HBM
// line by line, eight lanes to one request.  The rows advance together, `steps`
// segments at a time, and the table is emptied after each such part: the voxels
// of a part of eight fit it, where those of whole rows (22 000 of the head scan's 256 rows)
// would not.  A piece that finds no slot goes straight to HBM, and so do the later
// pieces of its lane in that part (a scan in acquisition order).
// 2e6 rows of 220 segments on the 256 x 256 x 64 grid, FP32 / FP64: sorted 5.04 /
// 4.72 ms (5.3 / 4.8 with the slots emptied one by one, and then 6.2 with lines of
// 4, 6.3 of 16; 18.0 / 18.0 with a table keyed by voxel for the whole row; 12.4 /
// 11.0 with that key in parts); acquisition order 17.5 / 18.0 ms (26.0 / 23.1;
// parts of 16 segments 20.5).
template <typename T>
struct BpTable {
    static constexpr int kLine = 8;       // consecutive voxels of a key
    static constexpr int kBits = sizeof(T) == 4 ? 10 : 9;
    static constexpr int kKeys = 1 << kBits;
    static constexpr int kSlots = kKeys * kLine;
    static constexpr int kProbes = 4;
};

template <typename T>
struct HashScatterSink {
    LdsPtr<int> keys;
    LdsPtr<T> vals;
    HbmPtr<T> g;
    double r;
    bool full;  // a probe sequence of this lane found no slot
    __device__ __forceinline__ void piece(int j, int, int, int, double c)
    {
        using B = BpTable<T>;
        const T v = T(r * c);
        const int line = j / B::kLine;
        unsigned s = (unsigned(line) * 2654435761u) >> (32 - B::kBits);
#pragma unroll 1
        for (int q = full ? B::kProbes : 0; q < B::kProbes; ++q) {
            int k = __hip_atomic_load(keys + s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (k == -1 && __hip_atomic_compare_exchange_strong(keys + s, &k, line, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                                __HIP_MEMORY_SCOPE_WORKGROUP))
                k = line;
            if (k == line) {
                __hip_atomic_fetch_add(vals + (s * B::kLine + unsigned(j) % B::kLine), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                return;
            }
            s = (s + 1) & (B::kKeys - 1);
        }
        full = true;
        __hip_atomic_fetch_add(g + j, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
};

template <typename T, bool HULL>
__global__ void __launch_bounds__(kWG) k_backproject(ProtonsDev p, int64_t first, int64_t n,
                                                     const T *__restrict__ rv, T *gout, int steps, const PathSrc src,
                                                     GridDev g, unsigned *status)
{
    using B = BpTable<T>;
    __shared__ int keys[B::kKeys];
    __shared__ T vals[B::kSlots];
    for (int q = threadIdx.x; q < B::kSlots; q += kWG) vals[q] = T(0);
    for (int q = threadIdx.x; q < B::kKeys; q += kWG) keys[q] = -1;
    const int64_t i = first + int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    bool active = i < n;
    double ri = 0.0;
    Rec r{};
    if (active) {
        ri = double(rv[i]);
        if (ri == 0.0) {
            active = false;
        } else {
            r = load_rec(p, i);
            if (!rec_finite(r) || !isfinite(ri)) {
                raise_status(status, PCT_DEV_NONFINITE);
                active = false;
                r = Rec{};
            }
        }
    }
    const RowPath<HULL> path(src, g, r);
    LaneWalk<HULL> walk(path, g, r);
    HashScatterSink<T> s{(LdsPtr<int>)keys, (LdsPtr<T>)vals, (HbmPtr<T>)gout, ri, false};
    const int K = active ? path.K : 0;
    for (int k0 = 0; __syncthreads_or(k0 < K); k0 += steps) {
        s.full = false;
        if (k0 < K) {
            walk.run(k0, min(k0 + steps, K), s);
            if (k0 + steps >= K) walk.finish(s);
        }
        __syncthreads();
        // (four keys and sums read before any is used: one after the other, a call of
        // few workgroups waits for LDS 32 times a part; eight of them take more
        // registers than four waves a SIMD have)
        constexpr int kFlush = 4;
        static_assert(B::kSlots % (kFlush * kWG) == 0);
        for (int q0 = threadIdx.x; q0 < B::kSlots; q0 += kFlush * kWG) {
            int key[kFlush];
            T sum[kFlush];
#pragma unroll
            for (int u = 0; u < kFlush; ++u) {
                key[u] = keys[(q0 + u * kWG) / B::kLine];
                sum[u] = vals[q0 + u * kWG];
            }
#pragma unroll
            for (int u = 0; u < kFlush; ++u) {
                const int q = q0 + u * kWG;
                if (key[u] < 0) continue;
                if (sum[u] != T(0)) atomicAdd(gout + (key[u] * B::kLine + q % B::kLine), sum[u]);
                vals[q] = T(0);
                if (q % B::kLine == 0) keys[q / B::kLine] = -1;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// DROP
// ---------------------------------------------------------------------------
// Block accumulator for the FP32 value type: one 64-bit word per voxel holding
// the number of block rows that touch the voxel (bits 63..44) and the sum of
// rho_i a_ij in fixed point with kFixBits fractional bits (two's complement in
// the low bits).  One integer add per piece updates both, and integer
// addition makes the block sum independent of the order of the adds.  The sum
// must stay below kSumMax = 2^(43 - kFixBits) in magnitude.  A contribution of
// kFixMax or more is clamped to it and raises PCT_DEV_ACC_RANGE, a NaN one
// counts as zero.  The binned schedule also bounds every voxel's block sum by
// the sum over the block's rows of their largest contribution and raises the
// bit when that bound reaches kSumMax.
constexpr int kFixBits = 28;
constexpr int kCntShift = 44;
constexpr double kFixScale = double(1u << kFixBits);
constexpr double kFixMax = double(1u << 12);
constexpr double kSumMax = double(1ull << (kCntShift - 1 - kFixBits));

__device__ __forceinline__ unsigned long long pack_contribution(double v, bool first, unsigned *status)
{
    if (!(fabs(v) < kFixMax)) {
        atomicOr(status, PCT_DEV_ACC_RANGE);
        if (v != v) v = 0.0;
        else v = fmin(fmax(v, -kFixMax), kFixMax);
    }
    // adding 1.5 2^52 rounds to a whole number (to nearest, ties to even) and
    // leaves it in the low bits: |v| 2^28 stays below 2^41
    constexpr double kShift = 6755399441055744.0;
    const long long q = __double_as_longlong(fma(v, kFixScale, kShift)) - __double_as_longlong(kShift);
    return static_cast<unsigned long long>(q) + (first ? (1ull << kCntShift) : 0ull);
}

__device__ __forceinline__ void unpack_accumulator(unsigned long long w, int &cnt, double &sum)
{
    const long long W = static_cast<long long>(w);
    const long long c = (W + (1ll << (kCntShift - 1))) >> kCntShift;
    const long long V = W - (c << kCntShift);
    cnt = int(c);
    sum = double(V) * (1.0 / kFixScale);
}

// Order-independent FP64 block sums (deterministic mode): each contribution
// v is split into hi = round(v 2^28) and lo = round((v - hi 2^-28) 2^72), the
// first part exact (v's bits above 2^-28), the second within 2^-73, and both
// are summed in 64-bit integers, so the block sum hi 2^-28 + lo 2^-72 does not
// depend on the order of the adds.  A contribution of 2^16 or more (NaN: 0)
// is clamped and raises PCT_DEV_ACC_RANGE, which keeps the sums of blocks
// below 2^19 rows inside 64 bits.
constexpr double kDetHiScale = 268435456.0;                 // 2^28
constexpr double kDetLoScale = 4722366482869645213696.0;    // 2^72
constexpr double kDetMax = 65536.0;                         // 2^16

__device__ __forceinline__ void det_add(long long *hi, long long *lo, int j, double v, unsigned *status)
{
    if (!(fabs(v) < kDetMax)) {
        atomicOr(status, PCT_DEV_ACC_RANGE);
        v = v != v ? 0.0 : fmin(fmax(v, -kDetMax), kDetMax);
    }
    const double qh = rint(v * kDetHiScale);
    const double r = v - qh * (1.0 / kDetHiScale);
    atomicAdd(reinterpret_cast<unsigned long long *>(hi) + j, static_cast<unsigned long long>(static_cast<long long>(qh)));
    atomicAdd(reinterpret_cast<unsigned long long *>(lo) + j, static_cast<unsigned long long>(llrint(r * kDetLoScale)));
}

__device__ __forceinline__ double det_sum(long long hi, long long lo)
{
    return double(hi) * (1.0 / kDetHiScale) + double(lo) * (1.0 / kDetLoScale);
}

// One piece of a row into the block's accumulation: FP32 packed word; FP64
// double atomic, or the integer pair when acc_lo is given; the row count once.
template <typename T>
__device__ __forceinline__ void scatter_one(void *acc, long long *acc_lo, int32_t *cnt, int j, double v, bool first,
                                            unsigned *status)
{
    if constexpr (sizeof(T) == 4) {
        atomicAdd(static_cast<unsigned long long *>(acc) + j, pack_contribution(v, first, status));
    } else {
        if (acc_lo)
            det_add(static_cast<long long *>(acc), acc_lo, j, v, status);
        else
            atomicAdd(static_cast<double *>(acc) + j, v);
        if (first) atomicAdd(cnt + j, 1);
    }
}

// Touched range of a block, on large volumes (kRangeVoxels): least and
// greatest voxel index its rows add to, for the block's commit.  A slot holds the
// range in parts, each of a share of the workgroups and in a line of its own:
// atomics on one line take 4 ns each (26 us for 3200 rows on one slot's words side
// by side), and to look first whether a word has to move costs a round trip.
constexpr int kRangeParts = 32, kRangeSlots = 4;
struct alignas(256) RangePart {
    int lo, hi;
};
static_assert(kRangeSlots * kRangeParts * sizeof(RangePart) <= kMaxPartials * sizeof(double), "in Layout::partial");

struct TouchedRange {
    int lo = INT_MAX, hi = -1;
    __device__ __forceinline__ void touch(int j)
    {
        lo = min(lo, j);
        hi = max(hi, j);
    }
    // All lanes of the wave call it.
    __device__ __forceinline__ void publish(RangePart *slot)
    {
#pragma unroll
        for (int off = kWave / 2; off > 0; off >>= 1) {
            lo = min(lo, __shfl_xor(lo, off, kWave));
            hi = max(hi, __shfl_xor(hi, off, kWave));
        }
        if ((threadIdx.x & (kWave - 1)) != 0 || hi < 0) return;
        RangePart *part = slot + blockIdx.x % kRangeParts;
        atomicMin(&part->lo, lo);
        atomicMax(&part->hi, hi);
    }
};
__device__ __forceinline__ void clear_range(RangePart *slot)
{
    if (threadIdx.x >= kRangeParts) return;
    slot[threadIdx.x].lo = INT_MAX;
    slot[threadIdx.x].hi = -1;
}
// The whole range of a slot; all lanes of the wave call it.
__device__ __forceinline__ void read_range(const RangePart *slot, int &lo, int &hi)
{
    lo = slot[threadIdx.x % kRangeParts].lo;
    hi = slot[threadIdx.x % kRangeParts].hi;
#pragma unroll
    for (int off = kRangeParts / 2; off > 0; off >>= 1) {
        lo = min(lo, __shfl_xor(lo, off, kWave));
        hi = max(hi, __shfl_xor(hi, off, kWave));
    }
}
// [j0, j1): both slots' ranges and what lies between.
__device__ __forceinline__ void both_ranges(const RangePart *a, const RangePart *b, int &j0, int &j1)
{
    int lo, hi;
    read_range(a, lo, hi);
    read_range(b, j0, j1);
    j0 = min(lo, j0);
    j1 = max(hi, j1) + 1;
}
__global__ void __launch_bounds__(kWave) k_clear_ranges(RangePart *slots)
{
    for (int k = 0; k < kRangeSlots; ++k) clear_range(slots + k * kRangeParts);
}

// Scatter of one row: acc_j += rho a_ij and s_j += 1 once per row.  FP32 value
// type: packed 64-bit accumulator; FP64: double accumulator (or the integer
// pair) plus int count.
template <typename T, int CHORD>
struct DropScatterSink {
    void *acc;
    long long *acc_lo;  // FP64 deterministic mode: low words of the integer pair
    int32_t *cnt;
    unsigned *status;
    Reentry re;
    double rho;
    __device__ __forceinline__ void piece(int j, int ix, int iy, int iz, double c)
    {
        c = round_chord<CHORD>(c);
        bool first;
        re.visit(j, ix, iy, iz, c, first);
        scatter_one<T>(acc, acc_lo, cnt, j, rho * c, first, status);
    }
};

// One lane per row, two walks (lanes = 1, and grids whose in-plane index does not
// fit the wave kernels' packed pair).
template <typename T, int CHORD, bool HULL>
__global__ void __launch_bounds__(kWG) k_drop_rows(ProtonsDev p, const float *__restrict__ b,
                                                   const T *__restrict__ x, void *acc, int32_t *cnt,
                                                   const PathSrc src,  GridDev g, int64_t lo,
                                                   int64_t hi, double lambda, unsigned *status, long long *acc_lo,
                                                   const int *halt)
{
    if (gate_closed(halt)) return;
    int64_t i = lo + int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    bool active = i < hi;
    Rec r{};
    double bi = 0.0;
    if (active) {
        r = load_rec(p, i);
        bi = double(b[i]);
        if (!rec_finite(r) || !isfinite(bi)) {
            raise_status(status, PCT_DEV_NONFINITE);
            active = false;
        }
    }
    if (!active) return;
    __shared__ Reentry::Lds lds;
    Reentry re(lds, r);
    DotSink<T, true, CHORD> s{x, &re};
    const bool onward = walk_row<HULL>(r, src, g, s);
    if (!onward || re.unsafe) raise_status(status, PCT_DEV_REENTRY);
    if (!(s.n2 > 0.0)) return;
    DropScatterSink<T, CHORD> sc{acc, acc_lo, cnt, status, Reentry(lds, r), lambda * (bi - s.sum()) / s.n2};
    walk_row<HULL>(r, src, g, sc);
}

// ---------------------------------------------------------------------------
// DROP block kernels, one wave (and workgroup) per row: the row's records in
// LDS (pct_walk.hpp), a pass over its pieces for a_i.x and ||a_i||^2, and the
// scatter, a second pass over the same records (fused and separate schedule)
// or stored by the first one (binned schedule).
// ---------------------------------------------------------------------------
template <int LPP>
__device__ __forceinline__ double group_sum(double v)
{
#pragma unroll
    for (int off = LPP / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Record of the block that workgroup w takes (hi: none).  XCD-aware: workgroup
// w runs on XCD w mod 8, so the rows are dealt to the eight XCDs in contiguous
// runs of the block (a multiple of eight is launched, the padding workgroups
// idle), and each XCD walks a band of neighbouring paths of an ordered block
// and finds their voxels in its own L2.
__device__ __forceinline__ int64_t row_of_workgroup(int w, int64_t lo, int64_t hi)
{
    const int64_t per_xcd = (hi - lo + 7) / 8;
    const int64_t q = int64_t(w % 8) * per_xcd + w / 8;
    return q < hi - lo ? lo + q : hi;
}

// a_i.x and ||a_i||^2 of a row.  Chords enter a_i.x as CT values.
template <typename CT, int CHORD, bool HULL, class XA>
__device__ __forceinline__ void row_dot(const RowPath<HULL> &p, RecWindow &win, int dom, const XA &xa, bool &have,
                                        RowShape &shape, double &dot, double &n2)
{
    double d = 0.0, s = 0.0;
    const int sy = p.g.n[0], sz = p.g.n[0] * p.g.n[1];
    row_pieces<HULL, CHORD>(p, win, dom, have, shape, [&](const RowPiece &q) {
        if (!q.real) return;
        d = fma(double(CT(q.c)), xa(q.ix + sy * q.iy + sz * q.iz), d);
        s = fma(q.c, fma(2.0, q.before, q.c), s);
    });
    dot = wave_sum(d);
    n2 = wave_sum(s);
}

// Both passes of the atomic schedules over row i.
template <typename T, int CHORD, bool HULL, class XA>
__device__ __forceinline__ void drop_row(const ProtonsDev &p, const float *__restrict__ b, const XA &xa, void *acc,
                                         long long *acc_lo, int32_t *cnt, const PathSrc &src, const GridDev &g,
                                         int64_t i, int span, double lambda, unsigned *status, RangePart *range)
{
    using CT = typename std::conditional<sizeof(T) == 4, float, double>::type;
    extern __shared__ double lds[];
    const Rec r = load_rec(p, i);
    const double bi = double(b[i]);
    if (!rec_finite(r) || !isfinite(bi)) {
        raise_status(status, PCT_DEV_NONFINITE);
        return;
    }
    const RowPath<HULL> path(src, g, r);
    const int dom = dominant_axis(r);
    RecWindow win(lds, src.nvmax, span);
    bool have = false;
    RowShape shape;
    double dot, n2;
    row_dot<CT, CHORD, HULL>(path, win, dom, xa, have, shape, dot, n2);
    if (!shape.onward || shape.cut) raise_status(status, PCT_DEV_REENTRY);
    if (!(n2 > 0.0)) return;
    const double rho = lambda * (bi - dot) / n2;
    const int sy = g.n[0], sz = g.n[0] * g.n[1];
    TouchedRange touched;
    row_pieces<HULL, CHORD>(path, win, dom, have, shape, [&](const RowPiece &q) {
        if (!q.real) return;
        const int j = q.ix + sy * q.iy + sz * q.iz;
        scatter_one<T>(acc, acc_lo, cnt, j, rho * double(CT(q.c)), q.first, status);
        if (range) touched.touch(j);
    });
    if (range) touched.publish(range);
}

// Separate schedule: the block kernel (k_drop_commit follows).
template <typename T, int CHORD, bool HULL>
__global__ void __launch_bounds__(kWave) k_drop_block(ProtonsDev p, const float *__restrict__ b,
                                                      const T *__restrict__ x, void *acc, int32_t *cnt,
                                                      const PathSrc src, GridDev g, int64_t lo, int64_t hi,
                                                      double lambda, unsigned *status, long long *acc_lo,
                                                      const int *halt, int span, RangePart *range)
{
    if (gate_closed(halt)) return;
    const int64_t i = row_of_workgroup(int(blockIdx.x), lo, hi);
    if (i >= hi) return;
    drop_row<T, CHORD, HULL>(p, b, PlainX<T>{x}, acc, acc_lo, cnt, src, g, i, span, lambda, status, range);
}

// ---------------------------------------------------------------------------
// Fused FP32 DROP sweep: the commit of block q-1 happens inside the launch of
// block q.
//
// Two copies of the iterate (X0 = the caller's x, X1 in the workspace) and
// three packed accumulators rotate with the block index q of the sweep:
//   base = X[q % 2] holds every block before q-1;  PK[(q-1) % 3] holds block
//   q-1's sums.  Block q reads  xbar_j = base_j + sum_j / s_j  (the committed
//   value of block q-1, computed on the fly) and scatters into PK[q % 3].
//   In the same launch, commit workgroups write X[(q+1) % 2] = base + update
//   where block q-1 or q-2 touched a voxel (the only places where the two
//   copies differ), over the volume or, on a large one, over the two blocks'
//   touched ranges (slots q-1 and q-2 of four; slot q+1 is cleared for the next
//   block), and clear PK[(q-2) % 3].  Nothing read in a launch is written in it, so no grid-wide
//   synchronisation is needed, and the commit's memory traffic overlaps the
//   walk.  A flush kernel ends the sweep.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float committed_value(float base, unsigned long long w)
{
    if (w == 0ull) return base;
    int c;
    double sum;
    unpack_accumulator(w, c, sum);
    return float(double(base) + sum / double(c));
}

struct LazyX {
    const float *__restrict__ base;
    const unsigned long long *__restrict__ pk;
    __device__ __forceinline__ double operator()(int j) const { return double(committed_value(base[j], pk[j])); }
};

// Range slots of a fused launch (nullptr: the commit goes over the volume).
struct FusedRanges {
    RangePart *cur;
    const RangePart *prev, *old;
    RangePart *reset;
};

__device__ __forceinline__ void commit_part(const float *__restrict__ base, float *__restrict__ next,
                                            const unsigned long long *__restrict__ pk_prev,
                                            unsigned long long *__restrict__ pk_old, const FusedRanges &range,
                                            int nvox, int wg, int n_wg)
{
    int j0 = 0, j1 = nvox;
    if (range.cur) {
        both_ranges(range.prev, range.old, j0, j1);
        j0 &= ~3;
        if (wg == 0) clear_range(range.reset);
    }
    const int stride = 4 * n_wg * int(blockDim.x);
    for (unsigned ju = j0 + 4 * (wg * int(blockDim.x) + int(threadIdx.x)); ju < unsigned(j1); ju += stride) {
        const int j = int(ju);
        const ulonglong2 p01 = *reinterpret_cast<const ulonglong2 *>(pk_prev + j);
        const ulonglong2 p23 = *reinterpret_cast<const ulonglong2 *>(pk_prev + j + 2);
        const ulonglong2 o01 = *reinterpret_cast<const ulonglong2 *>(pk_old + j);
        const ulonglong2 o23 = *reinterpret_cast<const ulonglong2 *>(pk_old + j + 2);
        const unsigned long long wp[4] = {p01.x, p01.y, p23.x, p23.y};
        const unsigned long long wo[4] = {o01.x, o01.y, o23.x, o23.y};
        // next differs from base only where block q-1 or q-2 touched a voxel
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int jj = j + e;
            if ((wp[e] | wo[e]) != 0ull && jj < nvox) next[jj] = committed_value(base[jj], wp[e]);
            if (wo[e] != 0ull) pk_old[jj] = 0ull;
        }
    }
}

constexpr int kCommitWG = 1024;  // commit workgroups (64 threads) per fused launch
static_assert(kCommitWG % 8 == 0, "row workgroups must start on XCD 0");

template <int CHORD, bool HULL>
__global__ void __launch_bounds__(kWave) k_drop_fused(ProtonsDev p, const float *__restrict__ b,
                                                      const float *__restrict__ base, float *__restrict__ next,
                                                      const unsigned long long *__restrict__ pk_prev,
                                                      unsigned long long *pk_cur, unsigned long long *pk_old,
                                                      FusedRanges range, const PathSrc src, GridDev g, int64_t lo,
                                                      int64_t hi, double lambda, unsigned *status, int nvox, int span)
{
    if (int(blockIdx.x) < kCommitWG) {
        commit_part(base, next, pk_prev, pk_old, range, nvox, int(blockIdx.x), kCommitWG);
        return;
    }
    const int64_t i = row_of_workgroup(int(blockIdx.x) - kCommitWG, lo, hi);
    if (i >= hi) return;
    drop_row<float, CHORD, HULL>(p, b, LazyX{base, pk_prev}, pk_cur, nullptr, nullptr, src, g, i, span, lambda,
                                 status, range.cur);
}

// Start of a fused sweep: X1 = x.
__global__ void __launch_bounds__(256) k_sweep_begin(const float *__restrict__ x, float *__restrict__ x1, int nvox)
{
    for (int j = int(blockIdx.x * blockDim.x + threadIdx.x); j < nvox; j += int(gridDim.x * blockDim.x)) x1[j] = x[j];
}

// End of a fused sweep of T blocks: x = X[T%2] + update of block T-1; clears
// the accumulators of blocks T-1 and T-2.  (Where neither touched a voxel, x holds
// its value.)
__global__ void __launch_bounds__(256) k_sweep_end(float *x, const float *src, unsigned long long *pk_last,
                                                   unsigned long long *pk_prev, const RangePart *last,
                                                   const RangePart *prev, int nvox)
{
    int j0 = 0, j1 = nvox;
    if (last) both_ranges(last, prev, j0, j1);
    for (unsigned ju = j0 + blockIdx.x * blockDim.x + threadIdx.x; ju < unsigned(j1); ju += gridDim.x * blockDim.x) {
        const int j = int(ju);
        const unsigned long long w = pk_last[j];
        x[j] = committed_value(src[j], w);
        if (w != 0ull) pk_last[j] = 0ull;
        if (pk_prev[j] != 0ull) pk_prev[j] = 0ull;
    }
}

// ---------------------------------------------------------------------------
// Binned FP32 schedule: the block's D-weighted back-projection is staged per
// slab of the block's dominant axis and summed in LDS, one workgroup per slab.
//
// Launch 1 (k_drop_bin) goes over each row's pieces once.  The pieces of a row
// in one slab follow each other, so piece k of (slab, row) has a bin entry of
// its own: the chord (FP32), the voxel's cell in the slab, and whether another
// entry follows, written with plain stores.  At the end the row's rho_i =
// lambda (b_i - a_i.x) / ||a_i||^2 is stored.  Pieces without a bin (a row whose
// dominant axis is not the block's, a path that turns back along it, more than
// kBinCap pieces of one row in one slab) take a second pass, which adds rho_i
// a_ij to a packed overflow accumulator with a global atomic and raises the
// block's overflow flag.
//
// Launch 2 (k_slab_commit) gives each slab (and z chunk) of the block's axis
// to one workgroup: it adds rho_i a_ij of the slab's bin entries, packed with
// the row count bit, into a dense LDS window of the slab (64-bit integer
// adds), adds the overflow words of the window when the flag is up, and
// commits x_j = x_j + sum_j / s_j for every voxel of the window the block
// touched.  The integer sums per voxel are the ones the atomic schedules form,
// so without compensation the result is bitwise theirs; slabs are disjoint, so
// the commit is a plain read-modify-write of x over exactly the touched voxels.
//
// Compensation (default): the commit keeps the rounding error of the FP32
// iterate in a second FP32 word per voxel (lo, zero at the start of a call),
// forms base = x_j + lo_j + sum_j / s_j in FP64 and stores x_j = fl32(base),
// lo_j = fl32(base - x_j).  The gathers read x_j (the FP32 high part); x_j is
// the iterate rounded once, whatever the number of commits.
// ---------------------------------------------------------------------------
constexpr int kSlabWG = 1024;  // threads of a slab-commit workgroup

// One bin entry: the voxel's cell in the slab (an index of the slab's (b, z)
// plane, all ones: none) and the chord.  The first entry of a (slab, row) holds
// the cell in its low cell_bits, the epoch of its block above them and the
// number of entries less one in the top two bits; the others hold the cell in
// 30 bits and whether the row meets the voxel for the first time in the top one.
// Every block of a sweep has its own epoch, so an entry that an earlier block
// left says so by itself and nothing is cleared between blocks (the commit
// spent 3 us of its 27 on it at 256 slabs x 6400 rows); epochs start again at 1,
// over cleared bins, when their bits run out.
constexpr unsigned kFirstBit = 0x80000000u, kNoCell = 0x3FFFFFFFu;
struct BinEntry {
    unsigned cell;
    float c;
};

struct BinsDev {
    BinEntry *e0;   // [slab][cap]: first entries
    BinEntry *ek;   // [kBinCap - 1][slab][cap]: entries 1..
    double *rho;    // [cap]: rho_i of each row of the block, kSkipRow for a skipped one
    float *rowmax;  // [cap]: largest |rho_i a_ij| of each row of the block
    int cap;        // rows per block the bins hold (a multiple of 16)
    int nslab;      // max(nx, ny)
    int cell_bits;
    unsigned epoch;  // of the block
    __device__ __forceinline__ unsigned no_cell() const { return (1u << cell_bits) - 1u; }
};

// Where the iterate lies while a binned call runs: the caller's x with the
// compensation words beside it, or, packed, both in the workspace as (x, lo)
// pairs with z fastest, so that a slab of either in-plane axis is made of runs
// along z and a commit touches one line where it would touch one per voxel.
// Strides are in voxels; a cell of a slab is its index along the other in-plane
// axis times cb plus its index along z times cz.
struct IterateDev {
    float *x;    // x, or the pairs
    float *lo;   // compensation words (not packed)
    int packed;  // 0 or 1
    int sx, sy, sz;
    __device__ __forceinline__ int at(int ix, int iy, int iz) const { return ix * sx + iy * sy + iz * sz; }
    __device__ __forceinline__ float value(int j) const { return x[size_t(j) << packed]; }
};
constexpr unsigned long long kSkipRow = 0x7FF8DEADDEADDEADull;  // a NaN no arithmetic forms

// Dominant in-plane axis of the block, from its first record's gantry angle.
// It only routes pieces (rows of the other axis go to the overflow words,
// whose integer sums are the same), so a single-precision hardware cosine
// serves, the same in every kernel of the block.
__device__ __forceinline__ int block_axis(const ProtonsDev &p, int64_t lo)
{
    const float c = __cosf(p.gantry[lo]);
    return c * c >= 0.5f ? 0 : 1;
}

// Exact quotient floor(j / d) for j < 2^31 and 1 <= d < 2^30, from an FP64
// product with inv = 1 / d: the product is within 2^-20 of j / d, so the
// truncated quotient is off by at most one and one remainder test corrects
// it (a handful of instructions instead of the integer division sequence).
__device__ __forceinline__ unsigned udiv_exact(unsigned j, unsigned d, double inv)
{
    unsigned q = unsigned(double(j) * inv);
    const int r = int(j - q * d);
    if (r < 0) --q;
    else if (r >= int(d)) ++q;
    return q;
}

// Bound by VALU issue: about 1600 instructions a row (records 270 per round of 64
// segments, pieces 80 per round of 64 records, 250 to read the record and form
// its frame), 17 us at 6400 rows, the rest latency at four waves a SIMD.  One
// wave per row: 35.2 us for a 6400-row block of the 256 x 256 x 64 scan and 18.9
// us for 3200 rows on 200 x 200 x 32, against 61.2 and 33.4 us with each lane
// walking a run of slabs of its own (3700 instructions a row, the lanes' segments
// clipped and set up one by one) and 45 us with the same lanes carrying their
// voxel from segment to segment (1400, but a wave took every branch a lane did).
// Registers stay at four waves a SIMD: held to five or six, spills cost more.
template <int CHORD, bool HULL>
__global__ void __launch_bounds__(kWave) k_drop_bin(ProtonsDev p, const float *__restrict__ b,
                                                    IterateDev it, BinsDev bins,
                                                    unsigned long long *ovf, int *ovf_flag, const PathSrc src,
                                                    GridDev g, int64_t lo, int64_t hi, double lambda,
                                                    unsigned *status, const int *halt, int span)
{
    if (gate_closed(halt)) return;
    extern __shared__ double lds[];
    const int64_t i = row_of_workgroup(int(blockIdx.x), lo, hi);
    if (i >= hi) return;
    const int lane = int(threadIdx.x), row = int(i - lo);
    const Rec r = load_rec(p, i);
    const double bi = double(b[i]);
    const bool finite = rec_finite(r) && isfinite(bi);
    double rho = 0.0, n2 = 0.0;
    float cmax = 0.f;
    if (finite) {
        const RowPath<HULL> path(src, g, r);
        const int dom = dominant_axis(r);
        RecWindow win(lds, src.nvmax, span);
        bool have = false;
        RowShape shape;
        const bool binned = dom == block_axis(p, lo);
        const unsigned cap = unsigned(bins.cap), slabs = unsigned(bins.nslab), own = unsigned(dom ? g.n[1] : g.n[0]);
        const int cb = it.packed ? g.n[2] : 1, cz = it.packed ? 1 : dom ? g.n[0] : g.n[1];
        const unsigned tag = bins.epoch << bins.cell_bits, none = bins.no_cell();
        double d = 0.0, s = 0.0;
        float cw = 0.f, xw = 0.f;  // chord and gather of the pass before, in flight
        bool spilled = !binned;
        row_pieces<HULL, CHORD>(path, win, dom, have, shape, [&](const RowPiece &q) {
            const float cf = q.real ? float(q.c) : 0.f;
            d = fma(double(cw), double(xw), d);
            cw = cf;
            xw = 0.f;
            if (q.real) {
                xw = it.value(it.at(q.ix, q.iy, q.iz));
                s = fma(q.c, fma(2.0, q.before, q.c), s);
                cmax = fmaxf(cmax, cf);
                spilled |= q.k >= kBinCap;
            }
            // a record that is no piece still takes its place among the entries
            if (binned && shape.onward && unsigned(q.k) < unsigned(kBinCap) && unsigned(q.slab) < own) {
                const unsigned cell = unsigned((dom ? q.ix : q.iy) * cb + q.iz * cz);
                const unsigned at = unsigned(q.slab) * cap + unsigned(row);
                BinEntry *to = q.k == 0 ? bins.e0 + at : bins.ek + (unsigned(q.k - 1) * slabs * cap + at);
                const unsigned word = q.k == 0 ? (q.real ? cell : none) | tag | unsigned(q.more) << 30
                                               : (q.real ? cell : kNoCell) | (q.first ? kFirstBit : 0u);
                *to = BinEntry{word, cf};
            }
        });
        d = fma(double(cw), double(xw), d);
        const double dot = wave_sum(d);
        n2 = wave_sum(s);
        if ((!shape.onward || shape.cut) && lane == 0) raise_status(status, PCT_DEV_REENTRY);
        rho = lambda * (bi - dot) / n2;
        const bool direct = !binned || !shape.onward;
        if (n2 > 0.0 && (direct || __any(spilled))) {
            row_pieces<HULL, CHORD>(path, win, dom, have, shape, [&](const RowPiece &q) {
                if (q.real && (direct || q.k >= kBinCap))
                    atomicAdd(ovf + it.at(q.ix, q.iy, q.iz),
                              pack_contribution(rho * double(float(q.c)), q.first, status));
            });
            if (lane == 0) *ovf_flag = 1;
        }
    } else if (lane == 0) {
        raise_status(status, PCT_DEV_NONFINITE);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) cmax = fmaxf(cmax, __shfl_xor(cmax, off, 64));
    if (lane == 0) {
        const bool skip = !(n2 > 0.0);
        bins.rho[row] = skip ? __longlong_as_double(static_cast<long long>(kSkipRow)) : rho;
        bins.rowmax[row] = skip ? 0.f : float(fabs(rho * double(cmax)));
    }
}

// Start of the epochs: no entry in any bin; at the start of a sweep (`flags`)
// the overflow flags zero too.
__global__ void __launch_bounds__(256) k_bins_begin(BinEntry *e0, size_t n, int *ovf_flag, int flags)
{
    const size_t t = size_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (flags && t < 2) ovf_flag[t] = 0;
    uint4 *c4 = reinterpret_cast<uint4 *>(e0);
    for (size_t q = t; q < n / 2; q += size_t(gridDim.x) * blockDim.x) c4[q] = make_uint4(0u, 0u, 0u, 0u);
}

__global__ void __launch_bounds__(256) k_zero_f32(float *v, int64_t n)
{
    for (int64_t q = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; q < n; q += int64_t(gridDim.x) * blockDim.x)
        v[q] = 0.f;
}

// Word j of an array below 4 GB, by a 32-bit byte offset.
template <typename W>
__device__ __forceinline__ W *word_at(float *base, unsigned j)
{
    return reinterpret_cast<W *>(reinterpret_cast<char *>(base) + j * unsigned(sizeof(W)));
}

// Commit of block [lo, lo + nb) of the binned schedule: workgroup (slab s,
// chunk) sums the slab's bins of a range of cells into its LDS window and
// commits the touched voxels.  Thread t takes rows t, t + kSlabWG, ... of the
// block: their first and second entries are read coalesced, all at once (a
// second entry that was not written is ignored; waiting for the first ones to
// ask for it costs a round trip), then the rare third and fourth ones.  For the
// commit each wave lists the touched cells of its share of the window, so that
// the quotients run with full lanes (a tenth of the cells is touched).
// Bound by its chain of dependent round trips (entries, window, x): 17.0 us for a
// 6400-row block on 256 slabs and 13.4 us for 3200 rows on 200, 4.7 us of it the
// launch.  Cleared bins by parity, second entries asked for after the first ones
// and quotients over all cells took 26.9 and 19.6 us.
constexpr int kRowsPerThread = 8;  // rows of a block per slab-commit thread
constexpr int kListCells = 8;      // window cells per lane and list
constexpr int kListBatch = 4;      // listed cells per lane whose x loads are in flight together
constexpr size_t kListBytes = size_t(kSlabWG) * kListCells * sizeof(unsigned short);
static_assert(kWinWords <= 65536, "listed cells are 16-bit");

template <bool PACKED>
__device__ __forceinline__ void slab_commit_body(const ProtonsDev &p, int64_t lo, int nb, const BinsDev &bins,
                                                 int par, unsigned long long *ovf, int *ovf_flag,
                                                 const IterateDev &it, const GridDev &g, int chunk, int chunks,
                                                 int comp, const int *stored_axis, unsigned *status)
{
    extern __shared__ unsigned long long win[];
    const int tid = int(threadIdx.x);
    const int s = int(blockIdx.x) / chunks, part = int(blockIdx.x) % chunks;
    const int axis = stored_axis ? *stored_axis : block_axis(p, lo);
    const int nlat = g.n[1 - axis], cells = nlat * g.n[2];
    const int c0 = part * chunk, nw = min(chunk, cells - c0);
    if (blockIdx.x == 0 && tid == 0) ovf_flag[1 - par] = 0;
    const bool work = s < g.n[axis] && nw > 0;
    BinEntry er[kRowsPerThread], es[kRowsPerThread];
    double rr[kRowsPerThread];
    const size_t rank = size_t(bins.nslab) * bins.cap;
    const BinEntry *e0 = bins.e0 + size_t(s) * bins.cap, *ek = bins.ek + size_t(s) * bins.cap;
#pragma unroll
    for (int m = 0; m < kRowsPerThread; ++m) {
        const int r = tid + m * kSlabWG;
        er[m] = es[m] = BinEntry{0u, 0.f};
        rr[m] = 0.0;
        if (work && r < nb) {
            er[m] = e0[r];
            es[m] = ek[r];
            rr[m] = bins.rho[r];
        }
    }
    if (blockIdx.x == 0) {
        // every voxel's block sum is bounded by the sum over the rows of their
        // largest contribution: past kSumMax a sum may have left the word's range
        __shared__ double wsum[kSlabWG / 64];
        double t = 0.0;
        for (int q = tid; q < nb; q += kSlabWG) t += double(bins.rowmax[q]);
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) t += __shfl_xor(t, off, 64);
        if ((tid & 63) == 0) wsum[tid >> 6] = t;
        __syncthreads();
        if (tid == 0) {
            double tot = 0.0;
            for (int w = 0; w < kSlabWG / 64; ++w) tot += wsum[w];
            if (!(tot < kSumMax)) atomicOr(status, PCT_DEV_ACC_RANGE);
        }
    }
    if (!work) return;
    // entries of the row less one; -1 for a row without any in this block
    auto more_of = [&](int m) {
        const bool none = ((er[m].cell & kNoCell) >> bins.cell_bits) != bins.epoch ||
                          static_cast<unsigned long long>(__double_as_longlong(rr[m])) == kSkipRow;
        return none ? -1 : int(er[m].cell >> 30);
    };
    // the window is cleared while the entries are in flight
    for (int q = tid; q < nw; q += kSlabWG) win[q] = 0ull;
    __syncthreads();
    auto add = [&](unsigned cell, float c, double rho, bool first) {
        const int q = int(cell) - c0;
        if (unsigned(q) < unsigned(nw)) atomicAdd(&win[q], pack_contribution(rho * double(c), first, status));
    };
    const unsigned none = bins.no_cell();
    static_assert(kBinCap == 4, "third and fourth entries below");
    constexpr int kHalf = kRowsPerThread / 2;
#pragma unroll
    for (int h = 0; h < kRowsPerThread; h += kHalf) {
        if (h * kSlabWG >= nb) break;
        BinEntry e2[kHalf], e3[kHalf];
#pragma unroll
        for (int m = 0; m < kHalf; ++m) {
            const int more = more_of(h + m);
            e2[m] = e3[m] = BinEntry{kNoCell, 0.f};
            if (more >= 2) e2[m] = ek[rank + (tid + (h + m) * kSlabWG)];
            if (more >= 3) e3[m] = ek[2 * rank + (tid + (h + m) * kSlabWG)];
        }
#pragma unroll
        for (int m = h; m < h + kHalf; ++m) {
            const int more = more_of(m);
            const unsigned cell = er[m].cell & none;
            if (more >= 0 && cell != none) add(cell, er[m].c, rr[m], true);
            if (more >= 1 && (es[m].cell & kNoCell) != kNoCell)
                add(es[m].cell & kNoCell, es[m].c, rr[m], (es[m].cell & kFirstBit) != 0u);
            __builtin_amdgcn_sched_barrier(0);  // (the adds kept apart: together they take hundreds of registers)
        }
#pragma unroll
        for (int m = 0; m < kHalf; ++m) {
            if ((e2[m].cell & kNoCell) != kNoCell)
                add(e2[m].cell & kNoCell, e2[m].c, rr[h + m], (e2[m].cell & kFirstBit) != 0u);
            if ((e3[m].cell & kNoCell) != kNoCell)
                add(e3[m].cell & kNoCell, e3[m].c, rr[h + m], (e3[m].cell & kFirstBit) != 0u);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    const bool of = ovf_flag[par] != 0;
    __syncthreads();
    // cell = outer * inner + rest
    const unsigned inner = unsigned(PACKED ? g.n[2] : nlat);
    const double inv_inner = PACKED ? g.inv_n[2] : g.inv_n[1 - axis];
    const int sb = axis == 0 ? it.sy : it.sx, base = s * (axis == 0 ? it.sx : it.sy);
    const unsigned s_outer = unsigned(PACKED ? sb : it.sz), s_inner = unsigned(PACKED ? it.sz : sb);
    auto voxel = [&](int q) {
        const unsigned cell = unsigned(c0 + q), outer = udiv_exact(cell, inner, inv_inner);
        return unsigned(base) + outer * s_outer + (cell - outer * inner) * s_inner;
    };
    const int lane = tid & 63;
    unsigned short *list = reinterpret_cast<unsigned short *>(win + chunk) + (tid >> 6) * (64 * kListCells);
    for (int q0 = 0; q0 < nw; q0 += kListCells * kSlabWG) {
        int listed = 0;
#pragma unroll
        for (int u = 0; u < kListCells; ++u) {
            const int q = q0 + tid + u * kSlabWG;
            unsigned long long w = q < nw ? win[q] : 0ull;
            if (of && q < nw) {
                const unsigned j = voxel(q);
                const unsigned long long o = ovf[j];
                if (o != 0ull) {
                    w += o;
                    win[q] = w;
                    ovf[j] = 0ull;
                }
            }
            const unsigned long long mask = __ballot(w != 0ull);
            if (w != 0ull) list[listed + __popcll(mask & ((1ull << lane) - 1ull))] = static_cast<unsigned short>(q);
            listed += __popcll(mask);
        }
        for (int i0 = 0; i0 < listed; i0 += 64 * kListBatch) {
            unsigned jv[kListBatch];
            unsigned long long wv[kListBatch];
            float xv[kListBatch], lv[kListBatch];
#pragma unroll
            for (int u = 0; u < kListBatch; ++u) {
                const int i = i0 + u * 64 + lane;
                wv[u] = 0ull;
                jv[u] = 0u;
                xv[u] = lv[u] = 0.f;
                if (i < listed) {
                    const int q = list[i];
                    wv[u] = win[q];
                    jv[u] = voxel(q);
                    if constexpr (PACKED) {
                        const float2 v = *word_at<float2>(it.x, jv[u]);
                        xv[u] = v.x;
                        lv[u] = v.y;
                    } else {
                        xv[u] = *word_at<float>(it.x, jv[u]);
                        if (comp) lv[u] = *word_at<float>(it.lo, jv[u]);
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < kListBatch; ++u) {
                if (i0 + u * 64 + lane >= listed) continue;
                if (comp) {
                    int c;
                    double sum;
                    unpack_accumulator(wv[u], c, sum);
                    const double v = double(xv[u]) + double(lv[u]) + sum / double(c);
                    const float h = float(v), l = float(v - double(h));
                    if constexpr (PACKED) {
                        *word_at<float2>(it.x, jv[u]) = make_float2(h, l);
                    } else {
                        *word_at<float>(it.x, jv[u]) = h;
                        *word_at<float>(it.lo, jv[u]) = l;
                    }
                } else if constexpr (PACKED) {
                    *word_at<float2>(it.x, jv[u]) = make_float2(committed_value(xv[u], wv[u]), 0.f);
                } else {
                    *word_at<float>(it.x, jv[u]) = committed_value(xv[u], wv[u]);
                }
            }
        }
    }
}

template <bool PACKED>
__global__ void __launch_bounds__(kSlabWG) k_slab_commit(ProtonsDev p, int64_t lo, int nb, BinsDev bins, int par,
                                                         unsigned long long *ovf, int *ovf_flag, IterateDev it,
                                                         GridDev g, int chunk, int chunks, int comp,
                                                         const int *stored_axis, unsigned *status, GateDev gt)
{
    if (gate_closed(gt.halt)) return;
    slab_commit_body<PACKED>(p, lo, nb, bins, par, ovf, ovf_flag, it, g, chunk, chunks, comp, stored_axis, status);
    gate_commit_end(gt);
}

// Copies of the iterate between the caller's order (x fastest) and (x, lo) pairs
// with z fastest, through a tile of kTile x kTile voxels of one (x, z) plane.
constexpr int kTile = 32;

__global__ void __launch_bounds__(256) k_pack_iterate(const float *__restrict__ x, float2 *__restrict__ pairs,
                                                      GridDev g)
{
    __shared__ float tile[kTile][kTile + 1];
    const int tx = int(threadIdx.x) % kTile, ty = int(threadIdx.x) / kTile;
    const int x0 = int(blockIdx.x) * kTile, z0 = int(blockIdx.z) * kTile;
    for (int iy = int(blockIdx.y); iy < g.n[1]; iy += int(gridDim.y)) {
        for (int q = ty; q < kTile; q += 8)
            if (x0 + tx < g.n[0] && z0 + q < g.n[2])
                tile[q][tx] = x[x0 + tx + int64_t(g.n[0]) * (iy + int64_t(g.n[1]) * (z0 + q))];
        __syncthreads();
        for (int q = ty; q < kTile; q += 8)
            if (x0 + q < g.n[0] && z0 + tx < g.n[2])
                pairs[(int64_t(iy) * g.n[0] + x0 + q) * g.n[2] + z0 + tx] = make_float2(tile[tx][q], 0.f);
        __syncthreads();
    }
}

__global__ void __launch_bounds__(256) k_unpack_iterate(float *__restrict__ x, const float2 *__restrict__ pairs,
                                                        GridDev g)
{
    __shared__ float tile[kTile][kTile + 1];
    const int tx = int(threadIdx.x) % kTile, ty = int(threadIdx.x) / kTile;
    const int x0 = int(blockIdx.x) * kTile, z0 = int(blockIdx.z) * kTile;
    for (int iy = int(blockIdx.y); iy < g.n[1]; iy += int(gridDim.y)) {
        for (int q = ty; q < kTile; q += 8)
            if (x0 + q < g.n[0] && z0 + tx < g.n[2])
                tile[q][tx] = pairs[(int64_t(iy) * g.n[0] + x0 + q) * g.n[2] + z0 + tx].x;
        __syncthreads();
        for (int q = ty; q < kTile; q += 8)
            if (x0 + tx < g.n[0] && z0 + q < g.n[2])
                x[x0 + tx + int64_t(g.n[0]) * (iy + int64_t(g.n[1]) * (z0 + q))] = tile[tx][q];
        __syncthreads();
    }
}

// Commit of one block: a dense, coalesced scan of the volume, or of the block's
// touched range (and clears the slot of the next block); voxels with a non-zero
// row count get x_j += acc_j / s_j and are reset.
template <typename T>
__device__ __forceinline__ void drop_commit_body(T *x, void *accv, int32_t *cnt, int nvox, long long *acc_lo,
                                                 const RangePart *range, RangePart *range_next)
{
    int j0 = 0, j1 = nvox;
    if (range) {
        read_range(range, j0, j1);
        ++j1;
        if (blockIdx.x == 0) clear_range(range_next);
    }
    const unsigned stride = gridDim.x * blockDim.x, at = blockIdx.x * blockDim.x + threadIdx.x;
    if constexpr (sizeof(T) == 4) {
        // four 64-bit words per thread (the accumulator has 4 words of padding
        // past the last voxel; untouched words are zero)
        unsigned long long *pk = static_cast<unsigned long long *>(accv);
        for (unsigned ju = (j0 & ~3) + 4 * at; ju < unsigned(j1); ju += 4 * stride) {
            const int j = int(ju);
            const ulonglong2 w01 = *reinterpret_cast<const ulonglong2 *>(pk + j);
            const ulonglong2 w23 = *reinterpret_cast<const ulonglong2 *>(pk + j + 2);
            const unsigned long long w[4] = {w01.x, w01.y, w23.x, w23.y};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (w[e] != 0ull) {
                    int c;
                    double sum;
                    unpack_accumulator(w[e], c, sum);
                    if (c > 0) x[j + e] = T(double(x[j + e]) + sum / double(c));
                    pk[j + e] = 0ull;
                }
            }
        }
        return;
    }
    for (unsigned ju = j0 + at; ju < unsigned(j1); ju += stride) {
        const int j = int(ju), c = cnt[j];
        if (c == 0) continue;
        if (acc_lo) {
            long long *hi = static_cast<long long *>(accv);
            x[j] = T(double(x[j]) + det_sum(hi[j], acc_lo[j]) / double(c));
            hi[j] = 0;
            acc_lo[j] = 0;
        } else {
            double *acc = static_cast<double *>(accv);
            x[j] = T(double(x[j]) + acc[j] / double(c));
            acc[j] = 0.0;
        }
        cnt[j] = 0;
    }
}

template <typename T>
__global__ void __launch_bounds__(kWG) k_drop_commit(T *x, void *accv, int32_t *cnt, int nvox, long long *acc_lo,
                                                     const RangePart *range, RangePart *range_next, GateDev gt)
{
    if (gate_closed(gt.halt)) return;
    drop_commit_body<T>(x, accv, cnt, nvox, acc_lo, range, range_next);
    gate_commit_end(gt);
}

// ---------------------------------------------------------------------------
// total variation
// ---------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ double tv_diffs(const T *__restrict__ x, const GridDev &g, int ix, int iy, int iz,
                                           int64_t v, double eps, double &dx, double &dy, double &dz)
{
    const int64_t sy = g.n[0], sz = int64_t(g.n[0]) * g.n[1];
    double xv = x[v];
    dx = ix + 1 < g.n[0] ? double(x[v + 1]) - xv : 0.0;
    dy = iy + 1 < g.n[1] ? double(x[v + sy]) - xv : 0.0;
    dz = iz + 1 < g.n[2] ? double(x[v + sz]) - xv : 0.0;
    return sqrt(dx * dx + dy * dy + dz * dz + eps * eps);
}

template <typename T>
__global__ void __launch_bounds__(kWG) k_tv(const T *__restrict__ x, GridDev g, double eps, T *grad,
                                            double *partial, int64_t nvox)
{
    __shared__ double red[kWG];
    double local = 0.0;
    const int64_t sy = g.n[0], sz = int64_t(g.n[0]) * g.n[1];
    for (int64_t v = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; v < nvox; v += int64_t(gridDim.x) * blockDim.x) {
        int ix = int(v % g.n[0]);
        int iy = int((v / g.n[0]) % g.n[1]);
        int iz = int(v / sz);
        double dx, dy, dz;
        double s = tv_diffs(x, g, ix, iy, iz, v, eps, dx, dy, dz);
        local += s;
        if (grad) {
            double gv = -(dx + dy + dz) / s;
            double ex, ey, ez;
            if (ix > 0) gv += (double(x[v]) - double(x[v - 1])) / tv_diffs(x, g, ix - 1, iy, iz, v - 1, eps, ex, ey, ez);
            if (iy > 0) gv += (double(x[v]) - double(x[v - sy])) / tv_diffs(x, g, ix, iy - 1, iz, v - sy, eps, ex, ey, ez);
            if (iz > 0) gv += (double(x[v]) - double(x[v - sz])) / tv_diffs(x, g, ix, iy, iz - 1, v - sz, eps, ex, ey, ez);
            grad[v] = T(gv);
        }
    }
    red[threadIdx.x] = local;
    __syncthreads();
    for (int s = kWG / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

__global__ void __launch_bounds__(kWG) k_sum_partials(const double *__restrict__ partial, int n, double *out)
{
    __shared__ double red[kWG];
    double local = 0.0;
    for (int q = threadIdx.x; q < n; q += kWG) local += partial[q];
    red[threadIdx.x] = local;
    __syncthreads();
    for (int s = kWG / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = red[0];
}

// ---------------------------------------------------------------------------
// region selection (Algorithm 1, step 2): stable compaction of the records
// whose entry and exit slices lie in [z_lo, z_hi].  Each of G workgroups owns
// a contiguous chunk of the input: count, exclusive scan of the G counts,
// then an ordered scatter (wave ballots) inside every chunk.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int slice_index(float v, const GridDev &g)
{
    const double d = double(v);
    if (!isfinite(d)) return -1;
    const double s = floor((d - g.lo[2]) / g.pitch[2]);
    return int(fmin(fmax(s, 0.0), double(g.n[2] - 1)));
}

__device__ __forceinline__ bool region_member(const ProtonsDev &p, int64_t i, const GridDev &g, int z_lo, int z_hi)
{
    const int a = slice_index(p.v_in[i], g);
    const int c = slice_index(p.v_out[i], g);
    return a >= z_lo && a <= z_hi && c >= z_lo && c <= z_hi;
}

constexpr int kSelWG = 256;

// histogram of |exit slice - entry slice|: LDS bins per workgroup, then one
// global atomic per non-empty bin
__global__ void __launch_bounds__(kSelWG) k_span_histogram(ProtonsDev p, int64_t n, GridDev g,
                                                            unsigned long long *hist)
{
    extern __shared__ unsigned int bins[];
    const int nz = g.n[2];
    for (int k = threadIdx.x; k < nz; k += kSelWG) bins[k] = 0u;
    __syncthreads();
    for (int64_t i = int64_t(blockIdx.x) * kSelWG + threadIdx.x; i < n; i += int64_t(gridDim.x) * kSelWG) {
        const int a = slice_index(p.v_in[i], g);
        const int c = slice_index(p.v_out[i], g);
        if (a >= 0 && c >= 0) atomicAdd(&bins[a > c ? a - c : c - a], 1u);
    }
    __syncthreads();
    for (int k = threadIdx.x; k < nz; k += kSelWG)
        if (bins[k]) atomicAdd(hist + k, static_cast<unsigned long long>(bins[k]));
}

__global__ void __launch_bounds__(kSelWG) k_region_count(ProtonsDev p, int64_t n, int64_t chunk, GridDev g,
                                                          int z_lo, int z_hi, long long *partial)
{
    __shared__ long long red[kSelWG / 64];
    const int64_t a = int64_t(blockIdx.x) * chunk;
    const int64_t e = min(n, a + chunk);
    long long c = 0;
    for (int64_t i = a + threadIdx.x; i < e; i += kSelWG) c += region_member(p, i, g, z_lo, z_hi) ? 1 : 0;
    for (int o = 32; o > 0; o >>= 1) c += __shfl_down(c, o, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        long long t = 0;
        for (int w = 0; w < kSelWG / 64; ++w) t += red[w];
        partial[blockIdx.x] = t;
    }
}

// exclusive scan of G <= kMaxPartials counts in place; total to *count
__global__ void __launch_bounds__(kSelWG) k_region_scan(long long *partial, int G, int64_t *count)
{
    __shared__ long long run[kSelWG];
    const int per = (G + kSelWG - 1) / kSelWG;
    const int a = int(threadIdx.x) * per;
    const int e = min(G, a + per);
    long long s = 0;
    for (int k = a; k < e; ++k) s += partial[k];
    run[threadIdx.x] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        long long acc = 0;
        for (int t = 0; t < kSelWG; ++t) {
            const long long v = run[t];
            run[t] = acc;
            acc += v;
        }
        if (count) *count = acc;
    }
    __syncthreads();
    long long acc = run[threadIdx.x];
    for (int k = a; k < e; ++k) {
        const long long v = partial[k];
        partial[k] = acc;
        acc += v;
    }
}

__global__ void __launch_bounds__(kSelWG) k_region_scatter(ProtonsDev p, const float *b, int64_t n, int64_t chunk,
                                                            GridDev g, int z_lo, int z_hi, const long long *partial,
                                                            ProtonsBufDev out, int64_t capacity, float *b_out)
{
    __shared__ int wave_cnt[kSelWG / 64];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int64_t a = int64_t(blockIdx.x) * chunk;
    const int64_t e = min(n, a + chunk);
    long long base = partial[blockIdx.x];
    for (int64_t t0 = a; t0 < e; t0 += kSelWG) {
        const int64_t i = t0 + threadIdx.x;
        const bool f = i < e && region_member(p, i, g, z_lo, z_hi);
        const unsigned long long mask = __ballot(f);
        if (lane == 0) wave_cnt[wave] = __popcll(mask);
        __syncthreads();
        int before = 0, total = 0;
        for (int w = 0; w < kSelWG / 64; ++w) {
            before += w < wave ? wave_cnt[w] : 0;
            total += wave_cnt[w];
        }
        const long long dst = base + before + __popcll(mask & ((1ull << lane) - 1ull));
        if (f && dst < capacity) {
            out.t_in[dst] = p.t_in[i];
            out.v_in[dst] = p.v_in[i];
            out.th_in[dst] = p.th_in[i];
            out.ph_in[dst] = p.ph_in[i];
            out.t_out[dst] = p.t_out[i];
            out.v_out[dst] = p.v_out[i];
            out.th_out[dst] = p.th_out[i];
            out.ph_out[dst] = p.ph_out[i];
            out.gantry[dst] = p.gantry[i];
            if (b_out) b_out[dst] = b[i];
        }
        base += total;
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// stored rows (precision form): trace once, sweep from the stored CSR rows
// ---------------------------------------------------------------------------
// Counting sink: merged pieces of a row.
struct CountSink {
    int32_t n;
    __device__ __forceinline__ void piece(int, int, int, int, double) { ++n; }
};

// Row lengths (after consecutive merge) into offsets[1..n].
template <bool HULL>
__global__ void __launch_bounds__(kWG) k_row_lengths(ProtonsDev p, int64_t n, long long *len_out,
                                                     const PathSrc src,  GridDev g,
                                                     unsigned *status)
{
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    Rec r = load_rec(p, i);
    CountSink cs{0};
    if (rec_finite(r)) {
        walk_row<HULL>(r, src, g, cs);
    } else {
        raise_status(status, PCT_DEV_NONFINITE);
    }
    len_out[i] = cs.n;
}

// chunk sums of v[0..n) (G chunks of `chunk` values)
__global__ void __launch_bounds__(kSelWG) k_chunk_sums(const long long *v, int64_t n, int64_t chunk,
                                                        long long *partial)
{
    __shared__ long long red[kSelWG / 64];
    const int64_t a = int64_t(blockIdx.x) * chunk;
    const int64_t e = min(n, a + chunk);
    long long c = 0;
    for (int64_t i = a + threadIdx.x; i < e; i += kSelWG) c += v[i];
    for (int o = 32; o > 0; o >>= 1) c += __shfl_down(c, o, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        long long t = 0;
        for (int w = 0; w < kSelWG / 64; ++w) t += red[w];
        partial[blockIdx.x] = t;
    }
}

// in-place inclusive scan of every chunk, offset by the chunk's exclusive base
__global__ void __launch_bounds__(kSelWG) k_chunk_scan(long long *v, int64_t n, int64_t chunk,
                                                        const long long *partial)
{
    __shared__ long long tile[kSelWG];
    const int64_t a = int64_t(blockIdx.x) * chunk;
    const int64_t e = min(n, a + chunk);
    long long base = partial[blockIdx.x];
    for (int64_t t0 = a; t0 < e; t0 += kSelWG) {
        const int64_t i = t0 + threadIdx.x;
        tile[threadIdx.x] = i < e ? v[i] : 0;
        __syncthreads();
        for (int d = 1; d < kSelWG; d <<= 1) {
            const long long add = int(threadIdx.x) >= d ? tile[threadIdx.x - d] : 0;
            __syncthreads();
            tile[threadIdx.x] += add;
            __syncthreads();
        }
        if (i < e) v[i] = base + tile[threadIdx.x];
        base += tile[kSelWG - 1];
        __syncthreads();
    }
}

// Stored chord formats.
template <int CT>
struct StoredChord;
template <>
struct StoredChord<PCT_CHORD_F32> {
    using type = float;
    __device__ static __forceinline__ float put(double c) { return float(c); }
    __device__ static __forceinline__ float get(float v) { return v; }
};
template <>
struct StoredChord<PCT_CHORD_F16> {
    using type = unsigned short;
    __device__ static __forceinline__ unsigned short put(double c)
    {
        // c is already an FP16 value: the conversion is exact
        return __half_as_ushort(__float2half(float(c)));
    }
    __device__ static __forceinline__ float get(unsigned short v) { return __half2float(__ushort_as_half(v)); }
};
template <>
struct StoredChord<PCT_CHORD_BF16> {
    using type = unsigned short;
    __device__ static __forceinline__ unsigned short put(double c)
    {
        // c is already a BF16 value: its float has 16 zero low bits
        return static_cast<unsigned short>(__float_as_uint(float(c)) >> 16);
    }
    __device__ static __forceinline__ float get(unsigned short v) { return __uint_as_float(unsigned(v) << 16); }
};

// Rows are built by parts: the workgroup's rows take kRowSteps segments together
// and leave their pieces in LDS, from where the lanes of a wave write them eight to
// a row.  (A lane that writes its pieces as it meets them has a request to HBM for
// each, and 64 lines of 64 rows open at a time.)  1e6
// FP16 rows of 290 pieces: 2.5 ms, of which the writes nothing, against 6.7.
constexpr int kRowSteps = 4;
constexpr int kRowStage = 13;  // pieces of a row and part with a place in LDS: three a segment, and the row's last

template <int CT>
struct RowStage {
    int j[kWG][kRowStage];
    typename StoredChord<CT>::type c[kWG][kRowStage];
    long long base[kWG];
    int n[kWG];
};

template <int CT>
struct RowSink {
    using S = StoredChord<CT>;
    RowStage<CT> *stage;
    int32_t *vox;
    typename S::type *ch;
    int64_t pos, end;
    Reentry re;
    double n2;
    int staged = 0;  // pieces since the last write
    __device__ __forceinline__ void piece(int j, int ix, int iy, int iz, double c)
    {
        c = round_chord<CT>(c);
        bool first;
        const double aprev = re.visit(j, ix, iy, iz, c, first);
        n2 += c * (2.0 * aprev + c);
        const int v = first ? int(unsigned(j) | 0x80000000u) : j;
        if (staged < kRowStage) {
            stage->j[threadIdx.x][staged] = v;
            stage->c[threadIdx.x][staged] = S::put(c);
        } else if (pos < end) {  // (steps longer than a voxel)
            vox[pos] = v;
            ch[pos] = S::put(c);
        }
        ++staged;
        ++pos;
    }
};

template <int CT, bool HULL>
__global__ void __launch_bounds__(kWG) k_rows_build(ProtonsDev p, int64_t n, const long long *__restrict__ offsets,
                                                    int32_t *vox, typename StoredChord<CT>::type *chord, double *n2,
                                                    const PathSrc src,  GridDev g,
                                                    unsigned *status)
{
    __shared__ Reentry::Lds lds;
    __shared__ RowStage<CT> stage;
    const int tid = int(threadIdx.x);
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + tid;
    const bool mine = i < n;
    Rec r{};
    bool active = false;
    if (mine) {
        r = load_rec(p, i);
        active = rec_finite(r);
        if (!active) {
            raise_status(status, PCT_DEV_NONFINITE);
            r = Rec{};
        }
    }
    const RowPath<HULL> path(src, g, r);
    LaneWalk<HULL> walk(path, g, r);
    RowSink<CT> rs{&stage, vox, chord, mine ? offsets[i] : 0, mine ? offsets[i + 1] : 0, Reentry(lds, r), 0.0};
    const int K = active ? path.K : 0;
    for (int k0 = 0; __syncthreads_or(k0 < K); k0 += kRowSteps) {
        const int64_t base = rs.pos;
        rs.staged = 0;
        if (k0 < K) {
            walk.run(k0, min(k0 + kRowSteps, K), rs);
            if (k0 + kRowSteps >= K) walk.finish(rs);
        }
        stage.base[tid] = base;
        stage.n[tid] = int(min(int64_t(min(rs.staged, kRowStage)), max(rs.end - base, int64_t(0))));
        __syncthreads();
        const int row0 = tid & ~(kWave - 1);
#pragma unroll 1
        for (int q0 = 0; q0 < kWave; q0 += 8) {
            const int row = row0 + q0 + (tid & (kWave - 1)) / 8, cnt = stage.n[row];
            const long long to = stage.base[row];
            for (int q = tid % 8; q < cnt; q += 8) {
                vox[to + q] = stage.j[row][q];
                chord[to + q] = stage.c[row][q];
            }
        }
    }
    if (!mine) return;
    if (active && (!walk.onward || rs.re.unsafe)) raise_status(status, PCT_DEV_REENTRY);
    if (rs.pos != rs.end) raise_status(status, PCT_DEV_ROW_OVERFLOW);  // offsets from other records
    n2[i] = rs.n2;
}

struct RowsDev {
    const long long *offsets;
    const int32_t *vox;
    const void *chord;
    const double *n2;
};

constexpr int kRowRegs = 8;  // pieces per lane kept in registers between the gather and the scatter

// Fused FP32 DROP block over stored rows, where the call names its lanes per row or
// the workspace holds no bins for its blocks: LPR lanes per row, 64 / LPR rows per
// one-wave workgroup; commit workgroups first (see k_drop_fused).
template <int CT, int LPR>
__global__ void __launch_bounds__(64) k_drop_rows_fused(RowsDev rows, const float *__restrict__ b,
                                                        const float *__restrict__ base, float *__restrict__ next,
                                                        const unsigned long long *__restrict__ pk_prev,
                                                        unsigned long long *pk_cur, unsigned long long *pk_old,
                                                        FusedRanges range, int64_t lo, int64_t hi, double lambda,
                                                        unsigned *status, int nvox)
{
    if (int(blockIdx.x) < kCommitWG) {
        commit_part(base, next, pk_prev, pk_old, range, nvox, int(blockIdx.x), kCommitWG);
        return;
    }
    using S = StoredChord<CT>;
    const typename S::type *__restrict__ chord = static_cast<const typename S::type *>(rows.chord);
    constexpr int RPW = 64 / LPR;
    const int lane = threadIdx.x;
    const int l = lane % LPR;
    const int64_t i = lo + int64_t(blockIdx.x - kCommitWG) * RPW + lane / LPR;
    bool active = i < hi;
    int64_t a = 0, e = 0;
    double bi = 0.0, n2 = 0.0;
    if (active) {
        a = rows.offsets[i];
        e = rows.offsets[i + 1];
        bi = double(b[i]);
        n2 = rows.n2[i];
        if (!isfinite(bi)) {
            if (l == 0) raise_status(status, PCT_DEV_NONFINITE);
            active = false;
        }
    }
    if (!active) e = a;
    const LazyX xa{base, pk_prev};
    int jr[kRowRegs];
    float cr[kRowRegs];
    double dot = 0.0;
    // a piece naming a voxel outside the grid (rows built for another
    // plan) is dropped: chord 0 and voxel 0
    bool bad = false;
#pragma unroll
    for (int k = 0; k < kRowRegs; ++k) {
        const int64_t q = a + l + int64_t(k) * LPR;
        jr[k] = 0;
        cr[k] = 0.f;
        if (q < e) {
            const int v = rows.vox[q];
            if ((v & 0x7FFFFFFF) < nvox) {
                jr[k] = v;
                cr[k] = S::get(chord[q]);
            } else {
                bad = true;
            }
        }
    }
#pragma unroll
    for (int k = 0; k < kRowRegs; ++k)
        if (a + l + int64_t(k) * LPR < e) dot += double(cr[k]) * xa(jr[k] & 0x7FFFFFFF);
    for (int64_t q = a + l + int64_t(kRowRegs) * LPR; q < e; q += LPR) {
        const int j = rows.vox[q] & 0x7FFFFFFF;
        if (j < nvox)
            dot += double(S::get(chord[q])) * xa(j);
        else
            bad = true;
    }
    if (bad) raise_status(status, PCT_DEV_BAD_ROW);
    dot = group_sum<LPR>(dot);
    TouchedRange touched;
    if (active && n2 > 0.0) {
        const double rho = lambda * (bi - dot) / n2;
#pragma unroll
        for (int k = 0; k < kRowRegs; ++k) {
            if (a + l + int64_t(k) * LPR < e) {
                const int j = jr[k] & 0x7FFFFFFF;
                atomicAdd(pk_cur + j, pack_contribution(rho * double(cr[k]), jr[k] < 0, status));
                if (range.cur) touched.touch(j);
            }
        }
        for (int64_t q = a + l + int64_t(kRowRegs) * LPR; q < e; q += LPR) {
            const int v = rows.vox[q];
            const int j = v & 0x7FFFFFFF;
            if (j >= nvox) continue;
            atomicAdd(pk_cur + j, pack_contribution(rho * double(S::get(chord[q])), v < 0, status));
            if (range.cur) touched.touch(j);
        }
    }
    if (range.cur) touched.publish(range.cur);
}

// First kernel of a stored-row block of the binned schedule, one wave per row:
// what k_drop_bin leaves in the bins, from pieces that are read.  A row goes by
// bins when its slabs follow each other in one direction along the block's axis
// and every slab's first piece is the row's first in its voxel; any other row,
// one of more than kBinRegs * 64 pieces, and pieces past kBinCap of a slab are
// added to the overflow words.  The block's axis is the one along which its first
// row covers more voxels; the row's wave leaves it for the commit.
// 3200 FP16 rows of 290 pieces on 200 x 200 x 32: 15.5 us and 13.9 for the commit,
// where adding every piece to HBM words (k_drop_rows_fused, 9.3e5 atomics on
// scattered words at 2.3e10 a second) takes 33.2.  Bound by its chain of round
// trips (offsets, pieces, gather) and 7.4 MB of entries.
constexpr int kBinRegs = 8;

template <int CT>
__global__ void __launch_bounds__(kWave) k_rows_bin(RowsDev rows, const float *__restrict__ b, IterateDev it,
                                                    BinsDev bins, unsigned long long *ovf, int *ovf_flag, int *axis_out,
                                                    GridDev g, int64_t lo, int64_t hi, double lambda, unsigned *status,
                                                    int nvox)
{
    using S = StoredChord<CT>;
    const typename S::type *__restrict__ chord = static_cast<const typename S::type *>(rows.chord);
    const int64_t i = row_of_workgroup(int(blockIdx.x), lo, hi);
    if (i >= hi) return;
    const int lane = int(threadIdx.x), row = int(i - lo);
    const long long a = rows.offsets[i], e = rows.offsets[i + 1], fa = rows.offsets[lo], fe = rows.offsets[lo + 1];
    const double bi = double(b[i]), n2 = rows.n2[i];
    const int len = int(min(e - a, 0x7FFFFFFFll));
    const bool finite = isfinite(bi);
    if (!finite && lane == 0) raise_status(status, PCT_DEV_NONFINITE);
    struct Voxel {
        int x, y, z;
    };
    auto decode = [&](int j) {
        const unsigned z = udiv_exact(unsigned(j), unsigned(g.n[0]) * unsigned(g.n[1]), g.inv_nxy);
        const unsigned in = unsigned(j) - z * (unsigned(g.n[0]) * unsigned(g.n[1]));
        const unsigned y = udiv_exact(in, unsigned(g.n[0]), g.inv_n[0]);
        return Voxel{int(in - y * unsigned(g.n[0])), int(y), int(z)};
    };
    int vr[kBinRegs];
    float cr[kBinRegs];
    bool bad = false;
#pragma unroll
    for (int k = 0; k < kBinRegs; ++k) {
        const int q = lane + k * kWave;
        vr[k] = 0;
        cr[k] = 0.f;
        if (finite && q < len) {
            vr[k] = rows.vox[a + q];
            cr[k] = S::get(chord[a + q]);
        }
    }
    int axis = 0;
    if (fe > fa) {
        const int j0 = rows.vox[fa] & 0x7FFFFFFF, j1 = rows.vox[fe - 1] & 0x7FFFFFFF;
        if (j0 < nvox && j1 < nvox) {
            const Voxel v0 = decode(j0), v1 = decode(j1);
            axis = abs(v1.x - v0.x) >= abs(v1.y - v0.y) ? 0 : 1;
        }
    }
    if (row == 0 && lane == 0) *axis_out = axis;
    const int cb = it.packed ? g.n[2] : 1, cz = it.packed ? 1 : axis ? g.n[0] : g.n[1];
    // piece by piece: the gather, and where slabs start
    float xr[kBinRegs];
    unsigned long long starts[kBinRegs + 1];
    double dot = 0.0;
    bool up = false, down = false, met = false;
    int before = -1;
#pragma unroll
    for (int k = 0; k < kBinRegs; ++k) {
        starts[k] = ~0ull;
        xr[k] = 0.f;
        if (!finite || k * kWave >= len) continue;
        const bool on = lane + k * kWave < len;
        int j = vr[k] & 0x7FFFFFFF;
        if (j >= nvox) {  // rows built for another plan: chord 0 and voxel 0
            bad = true;
            j = vr[k] = 0;
            cr[k] = 0.f;
        }
        const Voxel v = decode(j);
        if (on) xr[k] = it.value(it.at(v.x, v.y, v.z));
        const int slab = axis ? v.y : v.x, prev = lane_before(slab, before);
        const bool inner = on && (k > 0 || lane > 0);
        up |= inner && slab > prev;
        down |= inner && slab < prev;
        const bool start = !on || !inner || slab != prev;
        met |= on && start && vr[k] >= 0;
        starts[k] = __ballot(start);
        before = lane_value(slab, kWave - 1);
    }
    starts[kBinRegs] = ~0ull;
#pragma unroll
    for (int k = 0; k < kBinRegs; ++k)
        if (finite && lane + k * kWave < len) dot += double(cr[k]) * double(xr[k]);
    for (int q = lane + kBinRegs * kWave; finite && q < len; q += kWave) {
        const int j = rows.vox[a + q] & 0x7FFFFFFF;
        if (j < nvox) {
            const Voxel v = decode(j);
            dot += double(S::get(chord[a + q])) * double(it.value(it.at(v.x, v.y, v.z)));
        } else {
            bad = true;
        }
    }
    if (bad) raise_status(status, PCT_DEV_BAD_ROW);
    dot = group_sum<kWave>(dot);
    const bool skip = !finite || !(n2 > 0.0);
    const double rho = skip ? 0.0 : lambda * (bi - dot) / n2;
    if (lane == 0) {
        bins.rho[row] = skip ? __longlong_as_double(static_cast<long long>(kSkipRow)) : rho;
        bins.rowmax[row] = 0.f;  // sums of stored rows are not bounded
    }
    if (skip) return;
    const bool direct = len > kBinRegs * kWave || __any(met) || (__any(up) && __any(down));
    const unsigned cap = unsigned(bins.cap), slabs = unsigned(bins.nslab), tag = bins.epoch << bins.cell_bits;
    int run = 0;  // pieces of the slab that the round before ended in
    bool spilled = false;
#pragma unroll
    for (int k = 0; k < kBinRegs; ++k) {
        if (k * kWave >= len) continue;
        const unsigned long long below = starts[k] & (~0ull >> (kWave - 1 - lane));
        const unsigned long long above = lane == kWave - 1 ? 0ull : starts[k] & (~0ull << (lane + 1));
        const int rank = below != 0ull ? lane - (kWave - 1 - __clzll(below)) : run + lane;
        const int rest = starts[k + 1] != 0ull ? __ffsll(static_cast<long long>(starts[k + 1])) - 1 : kWave;
        const int more = above != 0ull ? __ffsll(static_cast<long long>(above)) - 2 - lane : kWave - 1 - lane + rest;
        run = starts[k] != 0ull ? 1 + __clzll(starts[k]) : run + kWave;
        if (lane + k * kWave >= len) continue;
        const Voxel v = decode(vr[k] & 0x7FFFFFFF);
        if (direct || rank >= kBinCap) {
            atomicAdd(ovf + it.at(v.x, v.y, v.z), pack_contribution(rho * double(cr[k]), vr[k] < 0, status));
            spilled = true;
            continue;
        }
        const unsigned p = unsigned(axis ? v.y : v.x) * cap + unsigned(row);
        const unsigned cell = unsigned((axis ? v.x : v.y) * cb + v.z * cz);
        BinEntry *to = rank == 0 ? bins.e0 + p : bins.ek + (unsigned(rank - 1) * slabs * cap + p);
        const unsigned word = rank == 0 ? cell | tag | unsigned(min(more, 3)) << 30
                                        : cell | (vr[k] < 0 ? kFirstBit : 0u);
        *to = BinEntry{word, cr[k]};
    }
    for (int q = lane + kBinRegs * kWave; q < len; q += kWave) {
        const int v = rows.vox[a + q], j = v & 0x7FFFFFFF;
        if (j >= nvox) continue;
        const Voxel w = decode(j);
        atomicAdd(ovf + it.at(w.x, w.y, w.z),
                  pack_contribution(rho * double(S::get(chord[a + q])), v < 0, status));
        spilled = true;
    }
    if (__any(spilled) && lane == 0) *ovf_flag = 1;
}

// ---------------------------------------------------------------------------
// within-block ordering: every block of consecutive records is sorted by
// (entry slice, t_in, input position) with a bitonic sort of packed 64-bit
// keys in LDS, one workgroup per block
// ---------------------------------------------------------------------------
__device__ __forceinline__ unsigned long long order_key(const ProtonsDev &p, int64_t i, int local, const GridDev &g)
{
    const unsigned slice = unsigned(slice_index(p.v_in[i], g) + 1);  // 0 for a non-finite v_in
    unsigned t = __float_as_uint(p.t_in[i]);
    t ^= (t & 0x80000000u) ? 0xFFFFFFFFu : 0x80000000u;               // order-preserving bits
    return (static_cast<unsigned long long>(slice & 0xFFFFu) << 48) | (static_cast<unsigned long long>(t) << 16) |
           static_cast<unsigned long long>(local);
}

__global__ void __launch_bounds__(kSelWG) k_order_blocks(ProtonsDev p, const float *b, int64_t n, int64_t block,
                                                          int p2, GridDev g, ProtonsBufDev out, float *b_out)
{
    extern __shared__ unsigned long long keys[];
    const int64_t lo = int64_t(blockIdx.x) * block;
    const int cnt = int(min(block, n - lo));
    for (int q = threadIdx.x; q < p2; q += kSelWG) keys[q] = q < cnt ? order_key(p, lo + q, q, g) : ~0ull;
    __syncthreads();
    for (int k = 2; k <= p2; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int q = threadIdx.x; q < p2; q += kSelWG) {
                const int r = q ^ j;
                if (r > q) {
                    const unsigned long long a = keys[q], c = keys[r];
                    const bool up = (q & k) == 0;
                    if ((a > c) == up) {
                        keys[q] = c;
                        keys[r] = a;
                    }
                }
            }
            __syncthreads();
        }
    }
    for (int q = threadIdx.x; q < cnt; q += kSelWG) {
        const int64_t src = lo + int64_t(keys[q] & 0xFFFFull);
        const int64_t dst = lo + q;
        out.t_in[dst] = p.t_in[src];
        out.v_in[dst] = p.v_in[src];
        out.th_in[dst] = p.th_in[src];
        out.ph_in[dst] = p.ph_in[src];
        out.t_out[dst] = p.t_out[src];
        out.v_out[dst] = p.v_out[src];
        out.th_out[dst] = p.th_out[src];
        out.ph_out[dst] = p.ph_out[src];
        out.gantry[dst] = p.gantry[src];
        if (b_out) b_out[dst] = b[src];
    }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
static inline char *wsb(void *ws) { return static_cast<char *>(ws); }

static inline unsigned grid_for(int64_t n) { return unsigned((n + kWG - 1) / kWG); }

int upload_table(const pct_plan &pl, void *ws, void *stream)
{
    hipStream_t s = static_cast<hipStream_t>(stream);
    Layout L = layout_for(pl.nvox, pl.K, PCT_F32);
    hipError_t e = hipMemcpyAsync(wsb(ws) + L.table, pl.table.data(), pl.table.size() * sizeof(double),
                                  hipMemcpyHostToDevice, s);
    if (e != hipSuccess) return e;
    e = hipMemsetAsync(wsb(ws) + L.hdr, 0, 256, s);
    if (e != hipSuccess) return e;
    // the DROP accumulators and row counts start at zero; every block leaves
    // them at zero again
    e = hipMemsetAsync(wsb(ws) + L.acc, 0, L.cnt - L.acc, s);
    if (e != hipSuccess) return e;
    e = hipMemsetAsync(wsb(ws) + L.cnt, 0, size_t(pl.nvox) * sizeof(int32_t), s);
    if (e != hipSuccess) return e;
    return hipStreamSynchronize(s);
}

int read_status(const pct_plan &pl, void *ws, int reset, uint32_t *bits, void *stream)
{
    hipStream_t s = static_cast<hipStream_t>(stream);
    Layout L = layout_for(pl.nvox, pl.K, PCT_F32);
    uint32_t v = 0;
    hipError_t e = hipMemcpyAsync(&v, wsb(ws) + L.hdr, sizeof(v), hipMemcpyDeviceToHost, s);
    if (e != hipSuccess) return e;
    e = hipStreamSynchronize(s);
    if (e != hipSuccess) return e;
    *bits = v;
    if (reset) {
        e = hipMemsetAsync(wsb(ws) + L.hdr, 0, sizeof(uint32_t), s);
        if (e != hipSuccess) return e;
        e = hipStreamSynchronize(s);
    }
    return e;
}

static GateDev gate_dev(void *ws, const Layout &L, bool on)
{
    int *hdr = reinterpret_cast<int *>(wsb(ws) + L.hdr);
    GateDev gt{};
    if (!on) return gt;
    gt.halt = hdr + kHdrHalt;
    gt.wg_done = reinterpret_cast<unsigned *>(hdr + kHdrGateCount);
    gt.cancel = hdr + kHdrCancel;
    gt.done = reinterpret_cast<long long *>(hdr + kHdrDone);
    gt.status = reinterpret_cast<unsigned *>(hdr + kHdrStatus);
    return gt;
}

int write_cancel(pct_plan &pl, void *ws, int32_t request)
{
    hipStream_t cs = nullptr;
    {
        std::lock_guard<std::mutex> lock(pl.mu);
        if (!pl.cancel_stream) {
            hipError_t e = hipStreamCreateWithFlags(&cs, hipStreamNonBlocking);
            if (e != hipSuccess) return e;
            pl.cancel_stream = cs;
        }
        cs = static_cast<hipStream_t>(pl.cancel_stream);
    }
    Layout L = layout_for(pl.nvox, pl.K, PCT_F32);
    int *word = reinterpret_cast<int *>(wsb(ws) + L.hdr) + kHdrCancel;
    hipError_t e = hipMemsetD32Async(reinterpret_cast<hipDeviceptr_t>(word), request != 0 ? 1 : 0, 1, cs);
    if (e != hipSuccess) return e;
    return hipStreamSynchronize(cs);
}

int read_progress(const pct_plan &pl, void *ws, int64_t *done, int *halted, void *stream)
{
    hipStream_t s = static_cast<hipStream_t>(stream);
    Layout L = layout_for(pl.nvox, pl.K, PCT_F32);
    int32_t h[kHdrDone + 2];
    hipError_t e = hipMemcpyAsync(h, wsb(ws) + L.hdr, sizeof(h), hipMemcpyDeviceToHost, s);
    if (e != hipSuccess) return e;
    e = hipStreamSynchronize(s);
    if (e != hipSuccess) return e;
    int64_t d;
    std::memcpy(&d, h + kHdrDone, sizeof(d));
    *done = d;
    *halted = h[kHdrHalt] != 0;
    return hipSuccess;
}

int launch_gate_reset(const pct_plan &pl, void *ws, void *stream)
{
    Layout L = layout_for(pl.nvox, pl.K, PCT_F32);
    hipLaunchKernelGGL(k_gate_begin, dim3(1), dim3(64), 0, static_cast<hipStream_t>(stream), gate_dev(ws, L, true));
    return hipGetLastError();
}

int launch_trace(const pct_plan &pl, const ProtonsDev &p, int64_t first, int64_t count, int32_t max_nnz,
                 int32_t *vox, double *chord, int32_t *nnz, void *ws, void *stream)
{
    hipStream_t s = static_cast<hipStream_t>(stream);
    Layout L = layout_for(pl.nvox, pl.K, PCT_F32);
    const PathSrc src = path_src(pl, wsb(ws) + L.table);
    unsigned *status = reinterpret_cast<unsigned *>(wsb(ws) + L.hdr) + kHdrStatus;
    if (src.hull)
        hipLaunchKernelGGL(k_trace<true>, dim3(grid_for(count)), dim3(kWG), 0, s, p, first, count, max_nnz, vox,
                           chord, nnz, src, grid_dev(pl.grid), status);
    else
        hipLaunchKernelGGL(k_trace<false>, dim3(grid_for(count)), dim3(kWG), 0, s, p, first, count, max_nnz, vox,
                           chord, nnz, src, grid_dev(pl.grid), status);
    return hipGetLastError();
}

// Launches of the one-lane-per-proton kernels, in pieces of at most 2^30
// workgroups (protons [first, first + count) per piece).
template <class F>
static void launch_pieces(int64_t n, F &&piece)
{
    const int64_t max_n = int64_t(kWG) << 30;
    for (int64_t first = 0; first < n; first += max_n) piece(first, std::min<int64_t>(n - first, max_n));
}

int launch_forward(const pct_plan &pl, const ProtonsDev &p, int64_t n, const void *x, int dtype, void *y,
                   void *nrm2, void *ws, void *stream)
{
    hipStream_t s = static_cast<hipStream_t>(stream);
    Layout L = layout_for(pl.nvox, pl.K, PCT_F32);
    const PathSrc src = path_src(pl, wsb(ws) + L.table);
    unsigned *status = reinterpret_cast<unsigned *>(wsb(ws) + L.hdr) + kHdrStatus;
    GridDev g = grid_dev(pl.grid);
    auto go = [&](auto hull, auto norm, auto value) {
        using T = decltype(value);
        launch_pieces(n, [&](int64_t first, int64_t cnt) {
            hipLaunchKernelGGL((k_forward<T, decltype(hull)::value, decltype(norm)::value>), dim3(grid_for(cnt)),
                               dim3(kWG), 0, s, p, first, first + cnt, static_cast<const T *>(x),
                               static_cast<T *>(y), static_cast<T *>(nrm2), src, g, status);
        });
    };
    auto typed = [&](auto hull, auto norm) {
        if (dtype == PCT_F64)
            go(hull, norm, 0.0);
        else
            go(hull, norm, 0.0f);
    };
    auto normed = [&](auto hull) {
        if (nrm2)
            typed(hull, std::true_type{});
        else
            typed(hull, std::false_type{});
    };
    if (src.hull)
        normed(std::true_type{});
    else
        normed(std::false_type{});
    return hipGetLastError();
}

int launch_backproject(const pct_plan &pl, const ProtonsDev &p, int64_t n, const void *r, int dtype, void *gout,
                       void *ws, void *stream)
{
    hipStream_t s = static_cast<hipStream_t>(stream);
    Layout L = layout_for(pl.nvox, pl.K, PCT_F32);
    const PathSrc src = path_src(pl, wsb(ws) + L.table);
    unsigned *status = reinterpret_cast<unsigned *>(wsb(ws) + L.hdr) + kHdrStatus;
    GridDev g = grid_dev(pl.grid);
    // parts of 32 segments for calls of few workgroups, which wait for every part's
    // barriers and never for HBM's atomics: 1e4 rows, FP32 / FP64, sorted on 256 x 256
    // x 64 418 / 419 us by parts of 8, 402 / 385 of 32, in acquisition order on 200 x
    // 200 x 32 555 / 499 and 390 / 341
    const int steps = n <= 16384 ? 32 : 8;
    auto go = [&](auto hull) {
        constexpr bool H = decltype(hull)::value;
        launch_pieces(n, [&](int64_t first, int64_t cnt) {
            if (dtype == PCT_F64)
                hipLaunchKernelGGL((k_backproject<double, H>), dim3(grid_for(cnt)), dim3(kWG), 0, s, p, first,
                                   first + cnt, static_cast<const double *>(r), static_cast<double *>(gout),
                                   steps, src, g, status);
            else
                hipLaunchKernelGGL((k_backproject<float, H>), dim3(grid_for(cnt)), dim3(kWG), 0, s, p, first,
                                   first + cnt, static_cast<const float *>(r), static_cast<float *>(gout),
                                   steps, src, g, status);
        });
    };
    if (src.hull)
        go(std::true_type{});
    else
        go(std::false_type{});
    return hipGetLastError();
}

// Profiling: a pool of event pairs per kernel kind; launches are sampled
// evenly so that at most kProfSamples pairs are recorded per call.
constexpr int kProfSamples = 512;

static hipError_t prof_prepare(pct_plan &pl)
{
    for (int k = 0; k < 2; ++k) {
        pl.prof_used[k] = 0;
        while (pl.prof_events[k].size() < size_t(2 * kProfSamples)) {
            hipEvent_t e;
            hipError_t err = hipEventCreate(&e);
            if (err != hipSuccess) return err;
            pl.prof_events[k].push_back(e);
        }
    }
    return hipSuccess;
}

static inline hipEvent_t prof_event(pct_plan &pl, int kind, int idx)
{
    return static_cast<hipEvent_t>(pl.prof_events[kind][idx]);
}

int profile_read(pct_plan &pl, double ms[2], int64_t launches[2])
{
    for (int k = 0; k < 2; ++k) {
        ms[k] = 0.0;
        launches[k] = pl.prof_used[k];
        for (int i = 0; i < pl.prof_used[k]; ++i) {
            hipEvent_t a = prof_event(pl, k, 2 * i), b = prof_event(pl, k, 2 * i + 1);
            hipError_t e = hipEventSynchronize(b);
            if (e != hipSuccess) return e;
            float t = 0.f;
            e = hipEventElapsedTime(&t, a, b);
            if (e != hipSuccess) return e;
            ms[k] += t;
        }
    }
    return hipSuccess;
}

void profile_release(pct_plan &pl)
{
    for (int k = 0; k < 2; ++k) {
        for (void *e : pl.prof_events[k]) (void)hipEventDestroy(static_cast<hipEvent_t>(e));
        pl.prof_events[k].clear();
        pl.prof_used[k] = 0;
    }
}

static_assert(kRowsPerThread * kSlabWG >= kBinMaxRows, "slab commit covers the largest binned block");

// Packed words of a slab-commit window: 128 KB of LDS (and 16 KB of lists) once
// the kernel is allowed that much dynamic LDS, else 40 KB.
static int slab_window_words()
{
    static const int words = [] {
        hipError_t e = hipSuccess;
        for (const void *f : {reinterpret_cast<const void *>(&k_slab_commit<false>),
                              reinterpret_cast<const void *>(&k_slab_commit<true>)})
            if (e == hipSuccess)
                e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize,
                                        int(kWinWords * sizeof(unsigned long long) + kListBytes));
        (void)hipGetLastError();
        return e == hipSuccess ? kWinWords : kWinWords * 5 / 16;
    }();
    return words;
}

// Workgroups of a block kernel over n rows: a multiple of eight (see
// row_of_workgroup).
static inline unsigned row_grid(int64_t n) { return unsigned(8 * ((n + 7) / 8)); }

// Block steps of a call from which the iterate is packed (see IterateDev).
constexpr int64_t kPackBlocks = 8;

void graph_release(pct_plan &pl)
{
    if (pl.graph_exec) (void)hipGraphExecDestroy(static_cast<hipGraphExec_t>(pl.graph_exec));
    pl.graph_exec = nullptr;
    pl.graph_key.clear();
    if (pl.capture_stream) (void)hipStreamDestroy(static_cast<hipStream_t>(pl.capture_stream));
    pl.capture_stream = nullptr;
    if (pl.cancel_stream) (void)hipStreamDestroy(static_cast<hipStream_t>(pl.cancel_stream));
    pl.cancel_stream = nullptr;
}

// Voxels from which a commit goes over its block's touched range, in the fused and
// in the separate schedule.  Over the volume / over ranges, us a block step: FP16
// rows by atomics, slab-ordered blocks of 250 on 256 x 256 x 64 19.4 / 13.8, of 400 x
// 128 31.9 / 20.4, on 512^3 535 / 211, blocks of one angle over all slices, 250 x 64
// 22.4 / 23.1, 3200 x 64 58.2 / 59.9, x 96 72.6 / 74.1; FP64 rows traced, slab-
// ordered 400 on 256 x 256 x 64 18.9 / 20.8, x 128 22.5 / 21.4, x 256 28.8 / 21.4,
// 512^3 179 / 61, in acquisition order 20.1 / 22.7, 23.0 / 25.9, 29.3 / 31.6 and 183 /
// 186.
constexpr int64_t kFusedRangeVoxels = int64_t(1) << 22, kRangeVoxels = int64_t(1) << 24;

// Slot k of the touched ranges, nullptr below `from` voxels.
static RangePart *range_slot(const pct_plan &pl, void *ws, int64_t from, int64_t k)
{
    if (pl.nvox < from) return nullptr;
    const Layout L = layout_for(pl.nvox, pl.K, PCT_F32);
    return reinterpret_cast<RangePart *>(wsb(ws) + L.partial) + (k % kRangeSlots) * kRangeParts;
}

// Buffers of the fused FP32 schedule: X[0] = x, X[1] in the workspace,
// accumulators PK[0..2], range slots R[0..3] (nullptr: none).
struct FusedBufs {
    float *X[2];
    unsigned long long *PK[3];
    RangePart *R[kRangeSlots];
    int nv;
    unsigned copy_grid;
};

static FusedBufs fused_bufs(const pct_plan &pl, void *ws, float *x)
{
    const Layout L = layout_for(pl.nvox, pl.K, PCT_F32);
    FusedBufs F;
    F.X[0] = x;
    F.X[1] = reinterpret_cast<float *>(wsb(ws) + L.x1);
    for (int k = 0; k < 3; ++k)
        F.PK[k] = reinterpret_cast<unsigned long long *>(wsb(ws) + L.acc + size_t(k) * L.acc_stride);
    for (int k = 0; k < kRangeSlots; ++k) F.R[k] = range_slot(pl, ws, kFusedRangeVoxels, k);
    F.nv = int(pl.nvox);
    F.copy_grid = unsigned(std::min<int64_t>(2048, (pl.nvox + 255) / 256));
    return F;
}

// Arguments of the launch at position q of a fused sweep (see k_drop_fused).
struct FusedStep {
    const float *base;
    float *next;
    const unsigned long long *pk_prev;
    unsigned long long *pk_cur, *pk_old;
    FusedRanges range;
};

static FusedStep fused_step(const FusedBufs &F, int64_t q)
{
    return FusedStep{F.X[q % 2],   F.X[(q + 1) % 2],  F.PK[(q + 2) % 3],
                     F.PK[q % 3], F.PK[(q + 1) % 3], {F.R[q % 4], F.R[(q + 3) % 4], F.R[(q + 2) % 4], F.R[(q + 1) % 4]}};
}

// One fused sweep over blocks [b0, b1): copy, one launch per block (launch_q
// enqueues the kernel of block [lo, hi) at position q), flush.  Profiling
// samples the per-block launches evenly.
template <class LaunchQ>
static void enqueue_fused(pct_plan &pl, const FusedBufs &F, int64_t b0, int64_t b1, int64_t block, int64_t n,
                          hipStream_t s, bool record_events, int64_t every, LaunchQ launch_q)
{
    hipLaunchKernelGGL(k_sweep_begin, dim3(F.copy_grid), dim3(256), 0, s, F.X[0], F.X[1], F.nv);
    if (F.R[0]) hipLaunchKernelGGL(k_clear_ranges, dim3(1), dim3(kWave), 0, s, F.R[0]);
    int64_t q = 0;
    for (int64_t t = b0; t < b1; ++t, ++q) {
        const int64_t lo = t * block;
        const int64_t hi = std::min<int64_t>(n, lo + block);
        const bool sample = record_events && (q % every == 0) && pl.prof_used[0] < kProfSamples;
        if (sample) (void)hipEventRecord(prof_event(pl, 0, 2 * pl.prof_used[0]), s);
        launch_q(s, q, lo, hi, fused_step(F, q));
        if (sample) {
            (void)hipEventRecord(prof_event(pl, 0, 2 * pl.prof_used[0] + 1), s);
            pl.prof_used[0]++;
        }
    }
    if (q > 0) {
        const int64_t last = q - 1;
        hipLaunchKernelGGL(k_sweep_end, dim3(F.copy_grid), dim3(256), 0, s, F.X[0], F.X[q % 2], F.PK[last % 3],
                           F.PK[(last + 2) % 3], F.R[last % 4], F.R[(last + 3) % 4], F.nv);
    }
}

// Whether a call's sweeps are recorded into a graph.  Recording costs about 6
// us a launch, replaying saves about 1 us a block step, and only of short ones
// (block steps of tens of us hide their launches): 63 FP64 steps of 3200 rows
// on the 64 x 64 x 4 grid, six sweeps: 7.5 ms replayed, 8.4 ms recorded and
// replayed, 7.8 ms launched; 782 binned steps of 6400 rows: 39.9 ms both ways, 4
// ms more the first time.  A call that can be cancelled is always recorded: its
// enqueue holds the plan's lock, which the request needs.
constexpr int kGraphSweeps = 4;
constexpr int64_t kLaunchSteps = 2048;

static bool graph_sweeps(const pct_drop_opts &o)
{
    if (o.flags & (PCT_DROP_NO_GRAPH | PCT_DROP_PROFILE)) return false;
    return (o.flags & PCT_DROP_CANCELLABLE) || o.n_iter >= kGraphSweeps ||
           (o.block_end - o.block_begin) * o.n_iter > kLaunchSteps;
}

// Runs n_iter sweeps: directly on the stream, or captured once into a HIP
// graph (cached on the plan for an identical launch key) and replayed.
template <class Sweep>
static int run_sweeps(pct_plan &pl, const std::vector<uint64_t> &key, bool use_graph, int n_iter, bool prof,
                      hipStream_t s, Sweep sweep)
{
    if (!use_graph) {
        for (int it = 0; it < n_iter; ++it) sweep(s, prof && it == n_iter - 1);
        return hipGetLastError();
    }
    if (!pl.graph_exec || pl.graph_key != key) {
        // recorded on a private stream (the caller's stream may be the null
        // stream, which cannot be captured); launched on the caller's stream
        if (pl.graph_exec) (void)hipGraphExecDestroy(static_cast<hipGraphExec_t>(pl.graph_exec));
        pl.graph_exec = nullptr;
        pl.graph_key.clear();
        if (!pl.capture_stream) {
            hipStream_t cs = nullptr;
            hipError_t e = hipStreamCreateWithFlags(&cs, hipStreamNonBlocking);
            if (e != hipSuccess) return e;
            pl.capture_stream = cs;
        }
        hipStream_t cs = static_cast<hipStream_t>(pl.capture_stream);
        hipError_t e = hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal);
        if (e != hipSuccess) return e;
        sweep(cs, false);
        hipGraph_t graph = nullptr;
        e = hipStreamEndCapture(cs, &graph);
        if (e != hipSuccess) return e;
        hipGraphExec_t exec = nullptr;
        e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
        (void)hipGraphDestroy(graph);
        if (e != hipSuccess) return e;
        pl.graph_exec = exec;
        pl.graph_key = key;
    }
    for (int it = 0; it < n_iter; ++it) {
        hipError_t e = hipGraphLaunch(static_cast<hipGraphExec_t>(pl.graph_exec), s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

static inline uint64_t bits_of(double v)
{
    uint64_t u;
    std::memcpy(&u, &v, sizeof(u));
    return u;
}

// ---- binned schedule, host side ----------------------------------------------
struct BinnedCall {
    bool ok = false;  // the workspace holds the slab bins of a block and a slab's window fits the LDS budget
    bool packed = false, comp = false;
    BinsDev bins{};
    IterateDev it{};
    size_t nrow = 0, win_lds = 0;
    unsigned epochs = 0;
    int chunk = 0, chunks = 0;
    int *ovf_flag = nullptr;
    unsigned long long *ovf = nullptr;
    unsigned *status = nullptr;
};

static BinnedCall binned_call(const pct_plan &pl, float *x, void *ws, size_t ws_bytes, int64_t block, int64_t steps,
                              bool comp)
{
    BinnedCall B;
    const Layout L = layout_for(pl.nvox, pl.K, PCT_F32);
    const int nslab = std::max(pl.grid.nx, pl.grid.ny);
    const int64_t cells = int64_t(nslab) * pl.grid.nz;
    int cell_bits = 1;  // of a slab's cells and the value that says none
    while ((int64_t(1) << cell_bits) <= cells) ++cell_bits;
    B.ok = nslab <= 8192 && block <= kBinMaxRows && pl.nvox < (int64_t(1) << 30) && cell_bits < 30 &&
           ws_bytes >= L.total + bin_bytes(block, nslab);
    if (!B.ok) return B;
    B.comp = comp;
    // the packed iterate costs two copies of the volume a call (about 8 us each
    // at 256 x 256 x 64) and saves the commits of x-dominant blocks their strided
    // lines (30 against 26 us each before the other changes to the commit)
    B.packed = steps >= kPackBlocks && pl.nvox < (int64_t(1) << 29);
    B.it.packed = B.packed ? 1 : 0;
    B.it.x = reinterpret_cast<float *>(B.packed ? static_cast<void *>(wsb(ws) + L.x1) : static_cast<void *>(x));
    B.it.lo = reinterpret_cast<float *>(wsb(ws) + L.lo);
    B.it.sx = B.packed ? pl.grid.nz : 1;
    B.it.sy = B.packed ? pl.grid.nx * pl.grid.nz : pl.grid.nx;
    B.it.sz = B.packed ? 1 : pl.grid.nx * pl.grid.ny;
    const int64_t cap = bin_rows(block);
    B.nrow = size_t(nslab) * size_t(cap);
    B.bins.e0 = reinterpret_cast<BinEntry *>(wsb(ws) + L.total);
    B.bins.ek = B.bins.e0 + B.nrow;
    B.bins.rho = reinterpret_cast<double *>(B.bins.ek + B.nrow * (kBinCap - 1));
    B.bins.rowmax = reinterpret_cast<float *>(B.bins.rho + cap);
    B.bins.cap = int(cap);
    B.bins.nslab = nslab;
    B.bins.cell_bits = cell_bits;
    B.epochs = (1u << (30 - cell_bits)) - 1u;
    B.chunk = int(std::min<int64_t>(cells, slab_window_words()));
    B.chunks = int((cells + B.chunk - 1) / B.chunk);
    B.win_lds = size_t(B.chunk) * sizeof(unsigned long long) + kListBytes;
    int *hdr = reinterpret_cast<int *>(wsb(ws) + L.hdr);
    B.ovf_flag = hdr + kHdrOvf;
    B.ovf = reinterpret_cast<unsigned long long *>(wsb(ws) + L.acc);
    B.status = reinterpret_cast<unsigned *>(hdr) + kHdrStatus;
    return B;
}

// One sweep.  bin(s, lo, hi, bins, parity, e0, e1) launches the block's first
// kernel, timed by the events when there are any; stored_axis: where that kernel
// leaves the block's axis, or nullptr (the records tell).
template <class Bin>
static void enqueue_binned(pct_plan &pl, const BinnedCall &B, const ProtonsDev &p, const pct_drop_opts &o, int64_t n,
                           hipStream_t s, bool record_events, int64_t every, const int *stored_axis,
                           const GateDev &gate, Bin &&bin)
{
    BinsDev bins = B.bins;
    const GridDev g = grid_dev(pl.grid);
    auto commit = B.packed ? &k_slab_commit<true> : &k_slab_commit<false>;
    int64_t seq = 0;
    for (int64_t t = o.block_begin; t < o.block_end; ++t, ++seq) {
        const int64_t lo = t * o.block;
        const int64_t hi = std::min<int64_t>(n, lo + o.block);
        const int par = int(seq & 1);
        bins.epoch = unsigned(seq % B.epochs) + 1u;
        if (bins.epoch == 1u)
            hipLaunchKernelGGL(k_bins_begin, dim3(unsigned(std::min<size_t>(1024, (B.nrow / 2 + 255) / 256 + 1))),
                               dim3(256), 0, s, bins.e0, B.nrow, B.ovf_flag, seq == 0 ? 1 : 0);
        // sampled blocks: both kernels timed by their own launch events
        const bool sample = record_events && (seq % every == 0) && pl.prof_used[0] < kProfSamples;
        hipEvent_t e[4] = {nullptr, nullptr, nullptr, nullptr};
        if (sample) {
            e[0] = prof_event(pl, 0, 2 * pl.prof_used[0]);
            e[1] = prof_event(pl, 0, 2 * pl.prof_used[0] + 1);
            e[2] = prof_event(pl, 1, 2 * pl.prof_used[1]);
            e[3] = prof_event(pl, 1, 2 * pl.prof_used[1] + 1);
            pl.prof_used[0]++;
            pl.prof_used[1]++;
        }
        bin(s, lo, hi, bins, par, e[0], e[1]);
        const dim3 grid(unsigned(bins.nslab * B.chunks));
        if (sample)
            hipExtLaunchKernelGGL(commit, grid, dim3(kSlabWG), uint32_t(B.win_lds), s, e[2], e[3], 0u, p, lo,
                                  int(hi - lo), bins, par, B.ovf, B.ovf_flag, B.it, g, B.chunk, B.chunks,
                                  B.comp ? 1 : 0, stored_axis, B.status, gate);
        else
            hipLaunchKernelGGL(commit, grid, dim3(kSlabWG), B.win_lds, s, p, lo, int(hi - lo), bins, par, B.ovf,
                               B.ovf_flag, B.it, g, B.chunk, B.chunks, B.comp ? 1 : 0, stored_axis, B.status, gate);
    }
}

// Around the sweeps of a call: the packed iterate formed and taken back, or the
// compensation words zeroed (they start at zero in every call, outside the graph).
static void binned_begin(const pct_plan &pl, const BinnedCall &B, float *x, hipStream_t s)
{
    const dim3 tiles(unsigned((pl.grid.nx + kTile - 1) / kTile), unsigned(std::min(pl.grid.ny, 65535)),
                     unsigned((pl.grid.nz + kTile - 1) / kTile));
    if (B.packed)
        hipLaunchKernelGGL(k_pack_iterate, tiles, dim3(256), 0, s, x, reinterpret_cast<float2 *>(B.it.x),
                           grid_dev(pl.grid));
    else if (B.comp)
        hipLaunchKernelGGL(k_zero_f32, dim3(unsigned(std::min<int64_t>(2048, (pl.nvox + 255) / 256))), dim3(256), 0, s,
                           B.it.lo, pl.nvox);
}
static int binned_end(const pct_plan &pl, const BinnedCall &B, float *x, hipStream_t s)
{
    if (!B.packed) return hipSuccess;
    const dim3 tiles(unsigned((pl.grid.nx + kTile - 1) / kTile), unsigned(std::min(pl.grid.ny, 65535)),
                     unsigned((pl.grid.nz + kTile - 1) / kTile));
    hipLaunchKernelGGL(k_unpack_iterate, tiles, dim3(256), 0, s, x, reinterpret_cast<const float2 *>(B.it.x),
                       grid_dev(pl.grid));
    return hipGetLastError();
}

template <typename T, int CHORD, bool HULL>
static int drop_loop(pct_plan &pl, const ProtonsDev &p, int64_t n, const float *b, T *x,
                     const pct_drop_opts &o, void *ws, size_t ws_bytes, hipStream_t s)
{
    const bool prof = (o.flags & PCT_DROP_PROFILE) != 0;
    if (prof) {
        hipError_t e = prof_prepare(pl);
        if (e != hipSuccess) return e;
    }
    // one lane per row on request, and where the wave kernels' records do not
    // hold the row; else a wave per row
    const int lanes = o.lanes == 1 || grid_dev(pl.grid).xy_shift == 0 || pl.K > kMaxRowSegments ? 1 : kWave;
    const int64_t nblk = o.block_end - o.block_begin;
    const int64_t every = std::max<int64_t>(1, (nblk + kProfSamples - 1) / kProfSamples);
    Layout L = layout_for(pl.nvox, pl.K, o.dtype);
    const PathSrc src = path_src(pl, wsb(ws) + L.table);
    const int span = record_span(pl.grid, pl.mlp.u_out - pl.mlp.u_in, std::min(src.nvmax, kMaxRowSegments + 3));
    const size_t rec_lds = record_bytes(src.nvmax, span);
    unsigned *status = reinterpret_cast<unsigned *>(wsb(ws) + L.hdr) + kHdrStatus;
    void *acc = wsb(ws) + L.acc;
    int32_t *cnt = reinterpret_cast<int32_t *>(wsb(ws) + L.cnt);
    GridDev g = grid_dev(pl.grid);
    const unsigned commit_grid = unsigned(std::min<int64_t>(4096, (pl.nvox + kWG - 1) / kWG));
    const bool cancellable = (o.flags & PCT_DROP_CANCELLABLE) != 0;
    const GateDev gate = gate_dev(ws, L, cancellable);
    // FP64 deterministic mode: integer block sums in the first two accumulators
    const bool det = sizeof(T) == 8 && (o.flags & PCT_DROP_DETERMINISTIC) != 0;
    long long *acc_lo = det ? reinterpret_cast<long long *>(wsb(ws) + L.acc + L.acc_stride) : nullptr;

    // Separate schedule: block kernel + commit per block.  (The one-lane kernel
    // leaves no ranges: its rows take far longer than the volume.)
    const bool ranges = lanes > 1 && pl.nvox >= kRangeVoxels;
    auto enqueue_sweep = [&](hipStream_t s, bool record_events) {
        int64_t seq = 0;
        if (ranges) hipLaunchKernelGGL(k_clear_ranges, dim3(1), dim3(kWave), 0, s, range_slot(pl, ws, kRangeVoxels, 0));
        for (int64_t t = o.block_begin; t < o.block_end; ++t, ++seq) {
            int64_t lo = t * o.block;
            int64_t hi = std::min<int64_t>(n, lo + o.block);
            RangePart *range = ranges ? range_slot(pl, ws, kRangeVoxels, seq) : nullptr;
            RangePart *range_next = ranges ? range_slot(pl, ws, kRangeVoxels, seq + 1) : nullptr;
            const bool sample = record_events && (seq % every == 0) && pl.prof_used[0] < kProfSamples;
            if (sample) (void)hipEventRecord(prof_event(pl, 0, 2 * pl.prof_used[0]), s);
            if (lanes == 1)
                hipLaunchKernelGGL((k_drop_rows<T, CHORD, HULL>), dim3(grid_for(hi - lo)), dim3(kWG), 0, s, p, b, x, acc,
                                   cnt, src, g, lo, hi, o.lambda, status, acc_lo, gate.halt);
            else
                hipLaunchKernelGGL((k_drop_block<T, CHORD, HULL>), dim3(row_grid(hi - lo)), dim3(kWave), rec_lds, s, p,
                               b, x, acc, cnt, src, g, lo, hi, o.lambda, status, acc_lo, gate.halt, span, range);
            if (sample) {
                (void)hipEventRecord(prof_event(pl, 0, 2 * pl.prof_used[0] + 1), s);
                pl.prof_used[0]++;
                (void)hipEventRecord(prof_event(pl, 1, 2 * pl.prof_used[1]), s);
            }
            hipLaunchKernelGGL(k_drop_commit<T>, dim3(commit_grid), dim3(kWG), 0, s, x, acc, cnt, int(pl.nvox),
                               acc_lo, range, range_next, gate);
            if (sample) {
                (void)hipEventRecord(prof_event(pl, 1, 2 * pl.prof_used[1] + 1), s);
                pl.prof_used[1]++;
            }
        }
    };
    BinnedCall B;  // FP32 default
    if (sizeof(T) == 4 && lanes > 1 && !(o.flags & (PCT_DROP_SEPARATE_COMMIT | PCT_DROP_FUSED_COMMIT)))
        B = binned_call(pl, reinterpret_cast<float *>(x), ws, ws_bytes, o.block, nblk * o.n_iter,
                        !(o.flags & PCT_DROP_NO_COMPENSATION));
    const bool binned = B.ok;
    const bool fused = sizeof(T) == 4 && lanes > 1 && !(o.flags & PCT_DROP_SEPARATE_COMMIT) && !binned && !cancellable;
    auto sweep = [&](hipStream_t s, bool record_events) {
        if constexpr (sizeof(T) == 4) {
            if (binned) {
                enqueue_binned(pl, B, p, o, n, s, record_events, every, nullptr, gate,
                               [&](hipStream_t s, int64_t lo, int64_t hi, const BinsDev &bins, int par, hipEvent_t e0,
                                   hipEvent_t e1) {
                                   const dim3 grid(row_grid(hi - lo));
                                   if (e0)
                                       hipExtLaunchKernelGGL((k_drop_bin<CHORD, HULL>), grid, dim3(kWave),
                                                             uint32_t(rec_lds), s, e0, e1, 0u, p, b, B.it, bins, B.ovf,
                                                             B.ovf_flag + par, src, g, lo, hi, o.lambda, status,
                                                             gate.halt, span);
                                   else
                                       hipLaunchKernelGGL((k_drop_bin<CHORD, HULL>), grid, dim3(kWave), rec_lds, s, p,
                                                          b, B.it, bins, B.ovf, B.ovf_flag + par, src, g, lo, hi,
                                                          o.lambda, status, gate.halt, span);
                               });
                return;
            }
            if (fused) {
                const FusedBufs F = fused_bufs(pl, ws, x);
                enqueue_fused(pl, F, o.block_begin, o.block_end, o.block, n, s, record_events, every,
                              [&](hipStream_t s, int64_t, int64_t lo, int64_t hi, const FusedStep &f) {
                                  hipLaunchKernelGGL((k_drop_fused<CHORD, HULL>),
                                                     dim3(kCommitWG + row_grid(hi - lo)), dim3(kWave), rec_lds, s,
                                                     p, b, f.base, f.next, f.pk_prev, f.pk_cur, f.pk_old, f.range, src, g, lo, hi,
                                                     o.lambda, status, F.nv, span);
                              });
                return;
            }
        }
        enqueue_sweep(s, record_events);
    };
    const bool use_graph = graph_sweeps(o);
    std::vector<uint64_t> key = {
        reinterpret_cast<uint64_t>(p.t_in),   reinterpret_cast<uint64_t>(p.v_in),
        reinterpret_cast<uint64_t>(p.th_in),  reinterpret_cast<uint64_t>(p.ph_in),
        reinterpret_cast<uint64_t>(p.t_out),  reinterpret_cast<uint64_t>(p.v_out),
        reinterpret_cast<uint64_t>(p.th_out), reinterpret_cast<uint64_t>(p.ph_out),
        reinterpret_cast<uint64_t>(p.gantry), reinterpret_cast<uint64_t>(b),
        reinterpret_cast<uint64_t>(x),        reinterpret_cast<uint64_t>(ws),
        uint64_t(n), uint64_t(o.block), uint64_t(o.block_begin), uint64_t(o.block_end),
        uint64_t(o.dtype), uint64_t(CHORD), uint64_t(lanes),
        uint64_t(fused) + 4 * uint64_t(binned) + 8 * uint64_t(B.comp) + 16 * uint64_t(cancellable) +
            32 * uint64_t(det) + 64 * uint64_t(B.packed),
        bits_of(o.lambda),
        0};
    if (cancellable) hipLaunchKernelGGL(k_gate_begin, dim3(1), dim3(64), 0, s, gate);
    if (binned) binned_begin(pl, B, reinterpret_cast<float *>(x), s);
    const int st = run_sweeps(pl, key, use_graph, o.n_iter, prof, s, sweep);
    if (!binned || st != hipSuccess) return st;
    return binned_end(pl, B, reinterpret_cast<float *>(x), s);
}

template <typename T>
static int drop_dispatch_chord(pct_plan &pl, const ProtonsDev &p, int64_t n, const float *b, T *x,
                               const pct_drop_opts &o, void *ws, size_t wsb_, hipStream_t s)
{
    auto go = [&](auto hull) -> int {
        constexpr bool H = decltype(hull)::value;
        switch (o.chord) {
        case PCT_CHORD_F32: return drop_loop<T, PCT_CHORD_F32, H>(pl, p, n, b, x, o, ws, wsb_, s);
        case PCT_CHORD_F16: return drop_loop<T, PCT_CHORD_F16, H>(pl, p, n, b, x, o, ws, wsb_, s);
        case PCT_CHORD_BF16: return drop_loop<T, PCT_CHORD_BF16, H>(pl, p, n, b, x, o, ws, wsb_, s);
        default: return drop_loop<T, PCT_CHORD_F64, H>(pl, p, n, b, x, o, ws, wsb_, s);
        }
    };
    return pl.hull ? go(std::true_type{}) : go(std::false_type{});
}

int launch_drop(pct_plan &pl, const ProtonsDev &p, int64_t n, const float *b, void *x, const pct_drop_opts &o,
                void *ws, size_t ws_bytes, void *stream)
{
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (o.dtype == PCT_F64)
        return drop_dispatch_chord<double>(pl, p, n, b, static_cast<double *>(x), o, ws, ws_bytes, s);
    return drop_dispatch_chord<float>(pl, p, n, b, static_cast<float *>(x), o, ws, ws_bytes, s);
}

int launch_span_histogram(const pct_plan &pl, const ProtonsDev &p, int64_t n, int64_t *hist, void *stream)
{
    hipStream_t s = static_cast<hipStream_t>(stream);
    const GridDev g = grid_dev(pl.grid);
    const unsigned grid = unsigned(std::max<int64_t>(1, std::min<int64_t>(2048, (n + kSelWG - 1) / kSelWG)));
    hipLaunchKernelGGL(k_span_histogram, dim3(grid), dim3(kSelWG), size_t(pl.grid.nz) * sizeof(unsigned), s, p, n, g,
                       reinterpret_cast<unsigned long long *>(hist));
    return hipGetLastError();
}

int launch_order_blocks(const pct_plan &pl, const ProtonsDev &p, int64_t n, const float *b, int64_t block,
                        const ProtonsBufDev &out, float *b_out, void *stream)
{
    hipStream_t s = static_cast<hipStream_t>(stream);
    int p2 = 2;
    while (p2 < block && p2 < n) p2 <<= 1;
    const int64_t nb = (n + block - 1) / block;
    hipLaunchKernelGGL(k_order_blocks, dim3(unsigned(nb)), dim3(kSelWG), size_t(p2) * sizeof(unsigned long long), s, p,
                       b, n, block, p2, grid_dev(pl.grid), out, b_out);
    return hipGetLastError();
}

int copy_device(void *dst, const void *src, size_t bytes, void *stream)
{
    return hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToDevice, static_cast<hipStream_t>(stream));
}

int launch_region_select(const pct_plan &pl, const ProtonsDev &p, int64_t n, const float *b, int z_lo, int z_hi,
                         const ProtonsBufDev &out, int64_t capacity, float *b_out, int64_t *count, void *ws,
                         void *stream)
{
    hipStream_t s = static_cast<hipStream_t>(stream);
    Layout L = layout_for(pl.nvox, pl.K, PCT_F32);
    long long *partial = reinterpret_cast<long long *>(wsb(ws) + L.partial);
    const GridDev g = grid_dev(pl.grid);
    const int64_t G = std::max<int64_t>(1, std::min<int64_t>(kMaxPartials, (n + kSelWG - 1) / kSelWG));
    int64_t chunk = (n + G - 1) / G;
    chunk = std::max<int64_t>(kSelWG, (chunk + kSelWG - 1) / kSelWG * kSelWG);
    hipLaunchKernelGGL(k_region_count, dim3(unsigned(G)), dim3(kSelWG), 0, s, p, n, chunk, g, z_lo, z_hi, partial);
    hipLaunchKernelGGL(k_region_scan, dim3(1), dim3(kSelWG), 0, s, partial, int(G), count);
    hipLaunchKernelGGL(k_region_scatter, dim3(unsigned(G)), dim3(kSelWG), 0, s, p, b, n, chunk, g, z_lo, z_hi,
                       partial, out, capacity, b_out);
    return hipGetLastError();
}

__global__ void k_zero_i64(long long *p, int64_t n)
{
    for (int64_t i = threadIdx.x; i < n; i += blockDim.x) p[i] = 0;
}

int launch_rows_count(const pct_plan &pl, const ProtonsDev &p, int64_t n, int64_t *offsets, void *ws, void *stream)
{
    hipStream_t s = static_cast<hipStream_t>(stream);
    Layout L = layout_for(pl.nvox, pl.K, PCT_F32);
    const PathSrc src = path_src(pl, wsb(ws) + L.table);
    unsigned *status = reinterpret_cast<unsigned *>(wsb(ws) + L.hdr) + kHdrStatus;
    long long *partial = reinterpret_cast<long long *>(wsb(ws) + L.partial);
    long long *off = reinterpret_cast<long long *>(offsets);
    hipLaunchKernelGGL(k_zero_i64, dim3(1), dim3(64), 0, s, off, int64_t(1));
    if (n > 0) {
        if (src.hull)
            hipLaunchKernelGGL(k_row_lengths<true>, dim3(grid_for(n)), dim3(kWG), 0, s, p, n, off + 1, src,
                               grid_dev(pl.grid), status);
        else
            hipLaunchKernelGGL(k_row_lengths<false>, dim3(grid_for(n)), dim3(kWG), 0, s, p, n, off + 1, src,
                               grid_dev(pl.grid), status);
        const int64_t G = std::max<int64_t>(1, std::min<int64_t>(kMaxPartials, (n + kSelWG - 1) / kSelWG));
        int64_t chunk = (n + G - 1) / G;
        chunk = std::max<int64_t>(kSelWG, (chunk + kSelWG - 1) / kSelWG * kSelWG);
        hipLaunchKernelGGL(k_chunk_sums, dim3(unsigned(G)), dim3(kSelWG), 0, s, off + 1, n, chunk, partial);
        hipLaunchKernelGGL(k_region_scan, dim3(1), dim3(kSelWG), 0, s, partial, int(G),
                           static_cast<int64_t *>(nullptr));
        hipLaunchKernelGGL(k_chunk_scan, dim3(unsigned(G)), dim3(kSelWG), 0, s, off + 1, n, chunk, partial);
    }
    return hipGetLastError();
}

int launch_rows_build(const pct_plan &pl, const ProtonsDev &p, int64_t n, int chord_type, const int64_t *offsets,
                      int32_t *vox, void *chord, double *n2, void *ws, void *stream)
{
    hipStream_t s = static_cast<hipStream_t>(stream);
    Layout L = layout_for(pl.nvox, pl.K, PCT_F32);
    const PathSrc src = path_src(pl, wsb(ws) + L.table);
    unsigned *status = reinterpret_cast<unsigned *>(wsb(ws) + L.hdr) + kHdrStatus;
    const long long *off = reinterpret_cast<const long long *>(offsets);
    const GridDev g = grid_dev(pl.grid);
    switch (chord_type) {
    case PCT_CHORD_F16:
        if (src.hull)
            hipLaunchKernelGGL((k_rows_build<PCT_CHORD_F16, true>), dim3(grid_for(n)), dim3(kWG), 0, s, p, n, off, vox,
                           static_cast<unsigned short *>(chord), n2, src, g, status);
        else
            hipLaunchKernelGGL((k_rows_build<PCT_CHORD_F16, false>), dim3(grid_for(n)), dim3(kWG), 0, s, p, n, off, vox,
                           static_cast<unsigned short *>(chord), n2, src, g, status);
        break;
    case PCT_CHORD_BF16:
        if (src.hull)
            hipLaunchKernelGGL((k_rows_build<PCT_CHORD_BF16, true>), dim3(grid_for(n)), dim3(kWG), 0, s, p, n, off, vox,
                           static_cast<unsigned short *>(chord), n2, src, g, status);
        else
            hipLaunchKernelGGL((k_rows_build<PCT_CHORD_BF16, false>), dim3(grid_for(n)), dim3(kWG), 0, s, p, n, off, vox,
                           static_cast<unsigned short *>(chord), n2, src, g, status);
        break;
    default:
        if (src.hull)
            hipLaunchKernelGGL((k_rows_build<PCT_CHORD_F32, true>), dim3(grid_for(n)), dim3(kWG), 0, s, p, n, off, vox,
                           static_cast<float *>(chord), n2, src, g, status);
        else
            hipLaunchKernelGGL((k_rows_build<PCT_CHORD_F32, false>), dim3(grid_for(n)), dim3(kWG), 0, s, p, n, off, vox,
                           static_cast<float *>(chord), n2, src, g, status);
    }
    return hipGetLastError();
}

template <int CT>
static void launch_rows_fused(int lanes, hipStream_t s, const RowsDev &rows, const float *b, const FusedStep &f,
                              int64_t lo, int64_t hi, double lambda, unsigned *status, int nvox)
{
    const int64_t n = hi - lo;
    switch (lanes) {
#define PCT_LAUNCH_ROWS(LPR)                                                                                     \
    case LPR: {                                                                                                  \
        const unsigned grid = unsigned(kCommitWG + (n + (64 / LPR) - 1) / (64 / LPR));                        \
        hipLaunchKernelGGL((k_drop_rows_fused<CT, LPR>), dim3(grid), dim3(64), 0, s, rows, b, f.base, f.next,     \
                           f.pk_prev, f.pk_cur, f.pk_old, f.range, lo, hi, lambda, status, nvox);                \
        break;                                                                                                   \
    }
        PCT_LAUNCH_ROWS(16)
        PCT_LAUNCH_ROWS(32)
        PCT_LAUNCH_ROWS(64)
#undef PCT_LAUNCH_ROWS
    default: break;
    }
}

// Whether a call's stored rows go by bins, the same sums as by atomics, so the same
// x.  Not where paths at 45 degrees have more pieces than k_rows_bin holds (the
// others go by overflow words, piece by piece, and its commit then reads the
// volume: rows of 650 pieces on 512 x 512 x 16 87 us a step of 3200 by bins, 69 by
// atomics, of 1030 on 800 x 800 x 16 204 and 160), and not where blocks are small
// for the volume, whose commit goes over all windows where that of the fused
// schedule goes over the block's range (slab-ordered blocks of 400 on 256 x 256 x 96
// 24.7 and 16.6 us, of 1000 x 256 44.0 and 33.8; blocks over all slices pay for that,
// 25.4 and 31.9, 43.6 and 101, which the call cannot tell).  Else whichever takes less: by bins
// two launches and work by the row, by atomics one launch and work by the piece and
// the voxel.  The costs are fitted (us a step, to about a tenth) to grids of 48 to
// 256 voxels across and 4 to 64 slices, blocks of 250 to 8000 rows of one angle; by
// bins / by atomics: 3200 rows on 200 x 200 x 32 27.9 / 31.8, 1600 22.4 / 17.1, 700
// 17.4 / 11.9; 8000 on 128 x 128 x 32 33.6 / 37.7, 3200 22.8 / 19.6; 8000 on 64 x 64
// x 64 29.1 / 20.9; 700 on 256 x 256 x 64 21.4 / 27.2.
static bool rows_by_bins(const pct_plan &pl, int64_t block)
{
    const pct_grid &g = pl.grid;
    const double depth = pl.mlp.u_out - pl.mlp.u_in, pitch = std::min(g.pitch[0], g.pitch[1]);
    const double most = std::min(M_SQRT2 * depth / pitch, double(g.nx) + double(g.ny)) +
                        std::min(0.03 * depth / g.pitch[2], double(g.nz));
    if (most > kBinRegs * kWave || block < pl.nvox / 12288) return false;
    const double pieces = 1.1 * std::min(depth, std::max(g.nx * g.pitch[0], g.ny * g.pitch[1])) / pitch;
    const double krows = 1e-3 * double(block), mvox = 1e-6 * double(pl.nvox);
    const double by_bins = 10.0 + 0.02 * std::max(g.nx, g.ny) + krows * (1.5 + 0.012 * pieces) + mvox;
    const double by_atomics = 4.0 + 0.034 * krows * pieces + 3.3 * mvox;
    return by_bins < by_atomics;
}

int launch_drop_rows(pct_plan &pl, const pct_rows &rows, const float *b, float *x, const pct_drop_opts &o, void *ws,
                     size_t ws_bytes, void *stream)
{
    hipStream_t s = static_cast<hipStream_t>(stream);
    const bool prof = (o.flags & PCT_DROP_PROFILE) != 0;
    if (prof) {
        hipError_t e = prof_prepare(pl);
        if (e != hipSuccess) return e;
    }
    const int lanes = o.lanes == 0 ? 64 : o.lanes;
    const int64_t nblk = o.block_end - o.block_begin;
    const int64_t every = std::max<int64_t>(1, (nblk + kProfSamples - 1) / kProfSamples);
    Layout L = layout_for(pl.nvox, pl.K, PCT_F32);
    unsigned *status = reinterpret_cast<unsigned *>(wsb(ws) + L.hdr) + kHdrStatus;
    const RowsDev rd{reinterpret_cast<const long long *>(rows.offsets), rows.vox, rows.chord, rows.n2};
    const int64_t n = rows.n;
    BinnedCall B;  // unless the call names its lanes per row
    if (o.lanes == 0 && rows_by_bins(pl, o.block)) B = binned_call(pl, x, ws, ws_bytes, o.block, nblk * o.n_iter, false);
    int *axis = reinterpret_cast<int *>(wsb(ws) + L.hdr) + kHdrAxis;
    const GridDev g = grid_dev(pl.grid);
    auto bin = [&](auto chord, hipStream_t s, int64_t lo, int64_t hi, const BinsDev &bins, int par, hipEvent_t e0,
                   hipEvent_t e1) {
        constexpr int CT = decltype(chord)::value;
        if (e0)
            hipExtLaunchKernelGGL(k_rows_bin<CT>, dim3(row_grid(hi - lo)), dim3(kWave), 0u, s, e0, e1, 0u, rd, b, B.it,
                                  bins, B.ovf, B.ovf_flag + par, axis, g, lo, hi, o.lambda, status, int(pl.nvox));
        else
            hipLaunchKernelGGL(k_rows_bin<CT>, dim3(row_grid(hi - lo)), dim3(kWave), 0, s, rd, b, B.it, bins, B.ovf,
                               B.ovf_flag + par, axis, g, lo, hi, o.lambda, status, int(pl.nvox));
    };
    auto sweep = [&](hipStream_t s, bool record_events) {
        if (B.ok) {
            enqueue_binned(pl, B, ProtonsDev{}, o, n, s, record_events, every, axis, GateDev{},
                           [&](hipStream_t s, int64_t lo, int64_t hi, const BinsDev &bins, int par, hipEvent_t e0,
                               hipEvent_t e1) {
                               if (rows.chord_type == PCT_CHORD_F16)
                                   bin(std::integral_constant<int, PCT_CHORD_F16>{}, s, lo, hi, bins, par, e0, e1);
                               else if (rows.chord_type == PCT_CHORD_BF16)
                                   bin(std::integral_constant<int, PCT_CHORD_BF16>{}, s, lo, hi, bins, par, e0, e1);
                               else
                                   bin(std::integral_constant<int, PCT_CHORD_F32>{}, s, lo, hi, bins, par, e0, e1);
                           });
            return;
        }
        const FusedBufs F = fused_bufs(pl, ws, x);
        enqueue_fused(pl, F, o.block_begin, o.block_end, o.block, n, s, record_events, every,
                      [&](hipStream_t s, int64_t, int64_t lo, int64_t hi, const FusedStep &f) {
                          switch (rows.chord_type) {
                          case PCT_CHORD_F16:
                              launch_rows_fused<PCT_CHORD_F16>(lanes, s, rd, b, f, lo, hi, o.lambda, status, F.nv);
                              break;
                          case PCT_CHORD_BF16:
                              launch_rows_fused<PCT_CHORD_BF16>(lanes, s, rd, b, f, lo, hi, o.lambda, status, F.nv);
                              break;
                          default:
                              launch_rows_fused<PCT_CHORD_F32>(lanes, s, rd, b, f, lo, hi, o.lambda, status, F.nv);
                          }
                      });
    };
    const bool use_graph = graph_sweeps(o);
    std::vector<uint64_t> key = {reinterpret_cast<uint64_t>(rows.offsets), reinterpret_cast<uint64_t>(rows.vox),
                                 reinterpret_cast<uint64_t>(rows.chord),   reinterpret_cast<uint64_t>(rows.n2),
                                 reinterpret_cast<uint64_t>(b),            reinterpret_cast<uint64_t>(x),
                                 reinterpret_cast<uint64_t>(ws),           uint64_t(n),
                                 uint64_t(o.block),                        uint64_t(o.block_begin),
                                 uint64_t(o.block_end),                    uint64_t(rows.chord_type),
                                 uint64_t(lanes),                          bits_of(o.lambda),
                                 uint64_t(B.ok) + 2 * uint64_t(B.packed), 1};
    if (B.ok) binned_begin(pl, B, x, s);
    const int st = run_sweeps(pl, key, use_graph, o.n_iter, prof, s, sweep);
    if (!B.ok || st != hipSuccess) return st;
    return binned_end(pl, B, x, s);
}

static int tv_into(const pct_plan &pl, const void *x, int dtype, double eps, double *value_dev, void *grad,
                   double *partial, hipStream_t s)
{
    int nblk = int(std::min<int64_t>(kMaxPartials, (pl.nvox + kWG - 1) / kWG));
    if (dtype == PCT_F64)
        hipLaunchKernelGGL(k_tv<double>, dim3(nblk), dim3(kWG), 0, s, static_cast<const double *>(x),
                           grid_dev(pl.grid), eps, static_cast<double *>(grad), partial, pl.nvox);
    else
        hipLaunchKernelGGL(k_tv<float>, dim3(nblk), dim3(kWG), 0, s, static_cast<const float *>(x),
                           grid_dev(pl.grid), eps, static_cast<float *>(grad), partial, pl.nvox);
    hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(kWG), 0, s, partial, nblk, value_dev);
    return hipGetLastError();
}

int launch_tv(const pct_plan &pl, const void *x, int dtype, double eps, double *value_dev, void *grad, void *ws,
              void *stream)
{
    const Layout L = layout_for(pl.nvox, pl.K, dtype);
    return tv_into(pl, x, dtype, eps, value_dev, grad, reinterpret_cast<double *>(wsb(ws) + L.partial),
                   static_cast<hipStream_t>(stream));
}

// TV without a workspace: the per-workgroup partial sums (at most
// kMaxPartials doubles, 32 KB) live in this file-scope device array, one copy
// per GPU, held until the process ends.  Host code never passes the array's
// name to a kernel: its device address is looked up once per device (with
// that device current) and kept.  Calls on one GPU share the array, so calls
// that overlap on one GPU race; every partial a call reads it has written
// first, so nothing needs clearing.
static __device__ __align__(256) double scratch[kMaxPartials];

constexpr int kMaxScratchDevices = 64;
static std::mutex g_scratch_mu;
static double *g_scratch[kMaxScratchDevices];

static hipError_t scratch_address(double **out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxScratchDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch[dev] = static_cast<double *>(p);
    }
    *out = g_scratch[dev];
    return hipSuccess;
}

int launch_tv_static(const pct_plan &pl, const void *x, int dtype, double eps, double *value_dev, void *grad,
                     void *stream)
{
    double *partial = nullptr;
    const hipError_t e = scratch_address(&partial);
    if (e != hipSuccess) return e;
    return tv_into(pl, x, dtype, eps, value_dev, grad, partial, static_cast<hipStream_t>(stream));
}

}  // namespace pct
