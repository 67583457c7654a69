// Device sort of an acquisition-order scan into angle bins.  Section IV-A of
// the paper reconstructs a scan taken with continuous gantry rotation; its
// records arrive in acquisition order and are grouped by angle bin, then by a
// slab of the entry height v_in, then by the lateral entry t_in, so that a
// block of consecutive records covers neighbouring paths.
//
// Each record gets a 64-bit key  a << (32 + bits_s) | s << 32 | ord(t_in)
// (ord: the FP32 bit pattern mapped so that unsigned order is numeric order,
// with -0 taken as +0; a non-finite record gets a = n_angles and sorts last),
// and the (key, position) pairs go through a least-significant-digit radix
// sort with 9-bit digits (8-bit ones for pairs that do not pack, and where the
// workspace has no room for 512 counts a tile), one pass per digit the key uses:
//
//   k_sort_keys         one thread per record: the key, and a packed 40-byte copy
//                       of the record (9 fields and b)
//   k_sort_hist         one workgroup per tile of 4608 pairs: digit counts in
//                       LDS, written digit-major (count of digit d in tile g at
//                       d * n_tiles + g), so that one exclusive scan of the
//                       counts gives every (digit, tile) its output offset
//   k_sort_count_*      that scan: partial sums of 4096 counts, then the scan of
//                       each segment from the sum of the partials before it
//   k_sort_scatter      one workgroup per tile, a wave per 576 pairs in input
//                       order: a lane's rank among the lanes of its wave with
//                       the same digit comes from 9 ballots (one per digit
//                       bit), the count of the wave's earlier pairs from LDS, so
//                       the waves meet only once, to add up their counts; equal
//                       digits keep their input order (stable).  The tile's pairs
//                       are staged in LDS in digit order and written out as one
//                       run per digit
//
// A pass needs only the digits to come: the first pass takes the position from
// the place and, where what is left of the key and the position fit 64 bits (a
// 45-bit key and 2^28 records do), the later ones move one word a record instead of
// a key and a position; the last writes the position alone.
//
//   k_sort_gather       one thread per output record: copy the record from its
//                       input position, read from the packed copy (the angles
//                       of a continuous scan are uniform in acquisition order,
//                       so sources are random: one or two cache lines per
//                       record instead of one per field)
//
// The sort is integer work: the output is unique and bit-exact whatever the
// launch shape.

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <type_traits>
#include <utility>

#include "pct_sort.h"

namespace pct {

namespace {

constexpr int kSortWG = 256;
constexpr int kRadixWG = 512;
constexpr int kRadixWaves = kRadixWG / 64;
constexpr int kSortRounds = 9;
constexpr int64_t kSortTile = int64_t(kRadixWG) * kSortRounds;  // records per tile
constexpr int64_t kCountTile = 2048;                            // the workspace has 256 counts for so many records
constexpr int kScanPer = 16;
constexpr int64_t kScanSeg = int64_t(kSortWG) * kScanPer;       // counts per scan workgroup
static_assert(kRadixWG * kSortRounds < 65536, "16-bit counts and places in a tile");

size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

__device__ inline unsigned long long sort_key(const SortDev &s, float phi32, float v32, float t32)
{
    if (!isfinite(phi32) || !isfinite(v32) || !isfinite(t32))
        return static_cast<unsigned long long>(s.n_angles) << (32 + s.bits_s);
    // angle bin: nearest bin centre a * dphi, taken modulo the turn (fa is an
    // integer, so the remainder is exact)
    const double fa = floor(double(phi32) / s.dphi + 0.5);
    double r = fmod(fa, double(s.n_angles));
    if (r < 0.0) r += double(s.n_angles);
    const unsigned a = unsigned(r);
    const double fs = floor((double(v32) - s.z0) / s.slab);
    const unsigned sl = fs <= 0.0 ? 0u : (fs >= double(s.n_slabs - 1) ? unsigned(s.n_slabs - 1) : unsigned(fs));
    unsigned u = __float_as_uint(t32 == 0.0f ? 0.0f : t32);
    u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
    return (static_cast<unsigned long long>(a) << (32 + s.bits_s)) | (static_cast<unsigned long long>(sl) << 32) |
           static_cast<unsigned long long>(u);
}

__global__ void __launch_bounds__(kSortWG) k_sort_keys(ProtonsDev p, const float *b, int64_t n, SortDev s,
                                                       unsigned long long *key, float *rec)
{
    // the workgroup's packed records are staged in LDS and written out as
    // 16-byte stores over its contiguous 10 * 256 floats
    __shared__ float4 stage[kSortWG * 10 / 4];
    float *st = reinterpret_cast<float *>(stage);
    const int64_t i0 = int64_t(blockIdx.x) * kSortWG;
    const int64_t i = i0 + threadIdx.x;
    if (i < n) {
        const float t = p.t_in[i], v = p.v_in[i], phi = p.gantry[i];
        key[i] = sort_key(s, phi, v, t);
        float *r = st + 10 * threadIdx.x;
        r[0] = t;
        r[1] = v;
        r[2] = p.th_in[i];
        r[3] = p.ph_in[i];
        r[4] = p.t_out[i];
        r[5] = p.v_out[i];
        r[6] = p.th_out[i];
        r[7] = p.ph_out[i];
        r[8] = phi;
        r[9] = b ? b[i] : 0.0f;
    }
    __syncthreads();
    const int count = int(min<int64_t>(kSortWG, n - i0));     // records of this workgroup
    const int nf = 10 * count;                                  // floats to write
    float *out = rec + 10 * i0;                                 // 16-byte aligned: 10 * 256 floats per workgroup
    for (int q = threadIdx.x; q < nf / 4; q += kSortWG) reinterpret_cast<float4 *>(out)[q] = stage[q];
    for (int q = (nf / 4) * 4 + threadIdx.x; q < nf; q += kSortWG) out[q] = st[q];
}

// Tile of a workgroup (n_tiles or more: none).  Workgroup w runs on XCD w mod 8, and
// what neighbouring tiles write lies side by side (their counts of a digit, their
// runs), so each XCD takes a contiguous run of tiles and its L2 fills the lines.
__device__ inline int64_t tile_of_workgroup(int64_t n_tiles)
{
    return int64_t(blockIdx.x % 8) * ((n_tiles + 7) / 8) + blockIdx.x / 8;
}
unsigned tile_grid(int64_t n_tiles) { return unsigned(8 * ((n_tiles + 7) / 8)); }

template <int BITS>
__global__ void __launch_bounds__(kRadixWG) k_sort_hist(const unsigned long long *key, int64_t n, int shift,
                                                        int64_t n_tiles, uint32_t *hist)
{
    constexpr int kDigits = 1 << BITS;
    static_assert(kDigits <= kRadixWG);
    __shared__ uint32_t h[kDigits];
    const int64_t tile = tile_of_workgroup(n_tiles), tile0 = tile * kSortTile;
    if (tile >= n_tiles) return;
    unsigned long long k[kSortRounds];
#pragma unroll
    for (int r = 0; r < kSortRounds; ++r) {
        const int64_t i = tile0 + int64_t(r) * kRadixWG + threadIdx.x;
        k[r] = i < n ? key[i] : 0ull;
    }
    if (threadIdx.x < kDigits) h[threadIdx.x] = 0;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSortRounds; ++r) {
        const int64_t i = tile0 + int64_t(r) * kRadixWG + threadIdx.x;
        if (i < n) atomicAdd(&h[unsigned(k[r] >> shift) & unsigned(kDigits - 1)], 1u);
    }
    __syncthreads();
    if (threadIdx.x < kDigits) hist[int64_t(threadIdx.x) * n_tiles + tile] = h[threadIdx.x];
}

// Exclusive prefix sum of v over a workgroup of WG threads in thread order; total
// gets the sum.  lds: WG / 64 words.
template <int WG>
__device__ inline uint32_t wg_exclusive_scan(uint32_t v, uint32_t *lds, uint32_t &total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t incl = v;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t a = __shfl_up(incl, off, 64);
        if (lane >= off) incl += a;
    }
    if (lane == 63) lds[wave] = incl;
    __syncthreads();
    uint32_t before = 0;
    total = 0;
    for (int w = 0; w < WG / 64; ++w) {
        const uint32_t c = lds[w];
        before += w < wave ? c : 0u;
        total += c;
    }
    __syncthreads();
    return before + incl - v;
}

__global__ void __launch_bounds__(kSortWG) k_sort_count_reduce(const uint32_t *hist, int64_t nh, uint32_t *part)
{
    __shared__ uint32_t lds[kSortWG / 64];
    const int64_t seg = int64_t(blockIdx.x) * kScanSeg;
    uint32_t sum = 0;
    for (int j = 0; j < kScanPer; ++j) {
        const int64_t e = seg + int64_t(j) * kSortWG + threadIdx.x;
        if (e < nh) sum += hist[e];
    }
    uint32_t total;
    wg_exclusive_scan<kSortWG>(sum, lds, total);
    if (threadIdx.x == 0) part[blockIdx.x] = total;
}

__global__ void __launch_bounds__(kSortWG) k_sort_count_down(uint32_t *hist, int64_t nh, const uint32_t *part)
{
    __shared__ uint32_t lds[kSortWG / 64];
    const int64_t first = int64_t(blockIdx.x) * kScanSeg + int64_t(threadIdx.x) * kScanPer;
    uint32_t v[kScanPer];
    uint32_t sum = 0, mine = 0;
    for (int j = 0; j < kScanPer; ++j) {
        const int64_t e = first + j;
        v[j] = e < nh ? hist[e] : 0u;
        sum += v[j];
    }
    for (unsigned q = threadIdx.x; q < blockIdx.x; q += kSortWG) mine += part[q];
    uint32_t base, total;
    wg_exclusive_scan<kSortWG>(mine, lds, base);
    uint32_t run = base + wg_exclusive_scan<kSortWG>(sum, lds, total);
    for (int j = 0; j < kScanPer; ++j) {
        const int64_t e = first + j;
        if (e < nh) hist[e] = run;
        run += v[j];
    }
}

// One pass.  PACKED: the pairs are words of the key's digits to come above the
// position (bits_n bits); idx_in is the place in the first pass (nullptr, raw
// keys) and not used in later ones, and the last pass (key_out nullptr) writes
// idx_out alone.  Otherwise key and position lie in two arrays, the position
// being the place in the first pass.
// Bound by its writes, runs of about eight words a digit: 56.7 us a pass of 1e7
// records (160 MB), 63.6 with the tiles dealt to the XCDs in turn, and 18.1 for the
// counts (23.3).  A 45-bit key takes five passes of 94 us; six of 8-bit digits,
// each moving a key and a position and ranking its waves together round by round,
// took 125 us each.
template <bool PACKED, int BITS>
__global__ void __launch_bounds__(kRadixWG) k_sort_scatter(const unsigned long long *key_in, const uint32_t *idx_in,
                                                           int64_t n, int shift, int bits_n, int64_t n_tiles,
                                                           const uint32_t *off, unsigned long long *key_out,
                                                           uint32_t *idx_out)
{
    constexpr int kDigits = 1 << BITS;
    __shared__ uint32_t first[kDigits];                           // output slot of the tile's first pair of each digit
    __shared__ uint32_t local[kDigits];                           // tile-local start of each digit (pairs in digit order)
    __shared__ volatile unsigned short cnt[kRadixWaves][kDigits]; // pairs of each wave and digit
    __shared__ unsigned long long skey[kSortTile];                // the tile's pairs, staged in digit order
    __shared__ unsigned short sdigit[PACKED ? kSortTile : 1];     // (a whole key tells)
    __shared__ uint32_t sidx[PACKED ? 1 : kSortTile];
    __shared__ uint32_t lds[kRadixWaves];
    const int t = threadIdx.x;
    const int lane = t & 63;
    const int wave = t >> 6;
    const int64_t tile = tile_of_workgroup(n_tiles);
    if (tile >= n_tiles) return;
    const int64_t i0 = tile * kSortTile + int64_t(wave) * (64 * kSortRounds) + lane;
    unsigned long long k[kSortRounds];
    uint32_t ix[kSortRounds], rank[kSortRounds];
#pragma unroll
    for (int r = 0; r < kSortRounds; ++r) {
        const int64_t i = i0 + 64 * r;
        k[r] = i < n ? key_in[i] : 0ull;
        ix[r] = uint32_t(i);
        if constexpr (!PACKED)
            if (idx_in && i < n) ix[r] = idx_in[i];
    }
    // pairs of digit t in this tile: the next offset of the scanned counts
    // (digit-major) minus this one; the last entry ends at n
    uint32_t mine = 0, tile_total;
    if (t < kDigits) {
        const int64_t e = int64_t(t) * n_tiles + tile;
        const uint32_t o0 = off[e];
        mine = (e + 1 < kDigits * n_tiles ? off[e + 1] : uint32_t(n)) - o0;
        first[t] = o0;
        for (int w = 0; w < kRadixWaves; ++w) cnt[w][t] = 0;
    }
    const uint32_t start = wg_exclusive_scan<kRadixWG>(mine, lds, tile_total);
    if (t < kDigits) local[t] = start;
    const unsigned long long below = (1ull << lane) - 1ull;
#pragma unroll
    for (int r = 0; r < kSortRounds; ++r) {
        const bool valid = i0 + 64 * r < n;
        const unsigned d = unsigned(k[r] >> shift) & unsigned(kDigits - 1);
        unsigned long long same = __ballot(valid);
#pragma unroll
        for (int bit = 0; bit < BITS; ++bit) {
            const unsigned long long m = __ballot((d >> bit) & 1u);
            same &= ((d >> bit) & 1u) ? m : ~m;
        }
        // LDS accesses of a wave are carried out in order: every lane reads the
        // count before the first lane of its digit raises it
        const uint32_t lower = uint32_t(__popcll(same & below)), seen = cnt[wave][d];
        rank[r] = seen + lower;
        if (valid && lower == 0) cnt[wave][d] = static_cast<unsigned short>(seen + uint32_t(__popcll(same)));
    }
    __syncthreads();
    if (t < kDigits) {
        uint32_t run = start;
        for (int w = 0; w < kRadixWaves; ++w) {
            const uint32_t c = cnt[w][t];
            cnt[w][t] = static_cast<unsigned short>(run);
            run += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSortRounds; ++r) {
        if (i0 + 64 * r >= n) continue;
        const unsigned long long rest = k[r] >> shift;
        const unsigned d = unsigned(rest) & unsigned(kDigits - 1);
        const uint32_t lp = cnt[wave][d] + rank[r];
        if (lp >= uint32_t(kSortTile)) continue;
        if constexpr (PACKED) {
            sdigit[lp] = static_cast<unsigned short>(d);
            const unsigned long long pos = shift == 0 ? static_cast<unsigned long long>(ix[r])
                                                      : k[r] & ((1ull << bits_n) - 1ull);
            skey[lp] = (rest >> BITS) << bits_n | pos;
        } else {
            skey[lp] = k[r];
            sidx[lp] = ix[r];
        }
    }
    __syncthreads();
    // write the staged pairs out in digit order: consecutive threads write
    // consecutive slots of each digit's run
    for (uint32_t q = uint32_t(t); q < tile_total && q < uint32_t(kSortTile); q += kRadixWG) {
        unsigned d;
        if constexpr (PACKED)
            d = sdigit[q];
        else
            d = unsigned(skey[q] >> shift) & unsigned(kDigits - 1);
        const uint32_t dst = first[d] + (q - local[d]);
        if (int64_t(dst) >= n) continue;
        if constexpr (PACKED) {
            if (key_out)
                key_out[dst] = skey[q];
            else
                idx_out[dst] = uint32_t(skey[q] & ((1ull << bits_n) - 1ull));
        } else {
            key_out[dst] = skey[q];
            idx_out[dst] = sidx[q];
        }
    }
}

__global__ void __launch_bounds__(kSortWG) k_sort_gather(const float *rec, int64_t n, const uint32_t *idx,
                                                         ProtonsBufDev o, float *b_out, int64_t *perm)
{
    const int64_t j = int64_t(blockIdx.x) * kSortWG + threadIdx.x;
    if (j >= n) return;
    const int64_t i = idx[j];
    if (i >= n) return;                 // idx is a permutation of 0 .. n-1
    const float2 *r = reinterpret_cast<const float2 *>(rec + 10 * i);
    const float2 r0 = r[0], r1 = r[1], r2 = r[2], r3 = r[3], r4 = r[4];
    o.t_in[j] = r0.x;
    o.v_in[j] = r0.y;
    o.th_in[j] = r1.x;
    o.ph_in[j] = r1.y;
    o.t_out[j] = r2.x;
    o.v_out[j] = r2.y;
    o.th_out[j] = r3.x;
    o.ph_out[j] = r3.y;
    o.gantry[j] = r4.x;
    if (b_out) b_out[j] = r4.y;
    if (perm) perm[j] = i;
}

}  // namespace

SortLayout sort_layout(int64_t n)
{
    SortLayout L{};
    L.n_tiles = (n + kSortTile - 1) / kSortTile;
    L.n_hist = 256 * ((n + kCountTile - 1) / kCountTile);
    L.n_parts = (L.n_hist + kScanSeg - 1) / kScanSeg;
    size_t o = 0;
    L.keys0 = o;
    o += align256(size_t(n) * 8);
    L.keys1 = o;
    o += align256(size_t(n) * 8);
    L.idx0 = o;
    o += align256(size_t(n) * 4);
    L.idx1 = o;
    o += align256(size_t(n) * 4);
    L.hist = o;
    o += align256(size_t(L.n_hist) * 4);
    L.part = o;
    o += align256(size_t(L.n_parts) * 4);
    L.rec = o;
    o += align256(size_t(n) * 40);
    L.total = o;
    return L;
}

int launch_sort_scan(const SortDev &s, const ProtonsDev &p, int64_t n, const float *b, const ProtonsBufDev &o,
                     float *b_out, int64_t *perm, void *ws, void *stream)
{
    if (n <= 0) return hipSuccess;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const SortLayout L = sort_layout(n);
    char *w = static_cast<char *>(ws);
    auto *k0 = reinterpret_cast<unsigned long long *>(w + L.keys0);
    auto *k1 = reinterpret_cast<unsigned long long *>(w + L.keys1);
    auto *i0 = reinterpret_cast<uint32_t *>(w + L.idx0);
    auto *i1 = reinterpret_cast<uint32_t *>(w + L.idx1);
    auto *hist = reinterpret_cast<uint32_t *>(w + L.hist);
    auto *part = reinterpret_cast<uint32_t *>(w + L.part);
    auto *rec = reinterpret_cast<float *>(w + L.rec);
    const unsigned blocks = unsigned((n + kSortWG - 1) / kSortWG);
    auto bits = [](uint64_t v) {
        int b = 0;
        for (; v != 0; v >>= 1) ++b;
        return b;
    };
    const int bits_n = bits(uint64_t(n - 1));
    auto sort = [&](auto packed_, auto bits_) {
        constexpr bool kPacked = decltype(packed_)::value;
        constexpr int kBits = decltype(bits_)::value;
        const int64_t nh = (int64_t(1) << kBits) * L.n_tiles;
        const unsigned parts = unsigned((nh + kScanSeg - 1) / kScanSeg), tiles = tile_grid(L.n_tiles);
        const int passes = (s.key_bits + kBits - 1) / kBits;
        for (int pass = 0; pass < passes; ++pass) {
            const int shift = !kPacked ? kBits * pass : pass > 0 ? bits_n : 0;
            hipLaunchKernelGGL(k_sort_hist<kBits>, dim3(tiles), dim3(kRadixWG), 0, st, k0, n, shift, L.n_tiles, hist);
            hipLaunchKernelGGL(k_sort_count_reduce, dim3(parts), dim3(kSortWG), 0, st, hist, nh, part);
            hipLaunchKernelGGL(k_sort_count_down, dim3(parts), dim3(kSortWG), 0, st, hist, nh, part);
            hipLaunchKernelGGL((k_sort_scatter<kPacked, kBits>), dim3(tiles), dim3(kRadixWG), 0, st, k0,
                               !kPacked && pass > 0 ? i0 : nullptr, n, shift, bits_n, L.n_tiles, hist,
                               kPacked && pass + 1 == passes ? nullptr : k1, i1);
            std::swap(k0, k1);
            std::swap(i0, i1);
        }
    };
    hipLaunchKernelGGL(k_sort_keys, dim3(blocks), dim3(kSortWG), 0, st, p, b, n, s, k0, rec);
    // one word a record where it holds what the first pass leaves of the key, and
    // the position; 512 counts a tile where the workspace has them (all but a
    // few sizes below 14336 records)
    using Eight = std::integral_constant<int, 8>;
    using Nine = std::integral_constant<int, 9>;
    const bool wide = 512 * L.n_tiles <= L.n_hist;
    if (bits_n == 0 || s.key_bits - (wide ? 9 : 8) + bits_n > 64)
        sort(std::false_type{}, Eight{});
    else if (wide)
        sort(std::true_type{}, Nine{});
    else
        sort(std::true_type{}, Eight{});
    hipLaunchKernelGGL(k_sort_gather, dim3(blocks), dim3(kSortWG), 0, st, rec, n, i0, o, b_out, perm);
    return hipGetLastError();
}

}  // namespace pct
