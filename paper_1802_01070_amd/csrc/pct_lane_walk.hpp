// Row walk of one lane: the polyline of one proton from segment to segment, for
// the kernels whose work is wide in rows (every lane has a row of its own, and
// the whole scan is one launch).
//
// The voxel of a vertex is known from the vertex alone, so a segment crosses
// the planes that lie between its two voxels and no others: at most one of each
// axis where the step is no longer than a voxel, and then the crossings are the
// at most three fractions of the segment, taken in ascending order.  The lanes
// of a wave take segment k together, so the coefficients of its vertex are
// scalar loads and only the number of crossings differs between lanes.
#pragma once

#include "pct_walk.hpp"

namespace pct {

// The walk.  run() takes the segments [k0, k1) and hands every finished piece
// that lies in the grid to sink.piece(j, ix, iy, iz, chord), consecutive parts
// in a voxel as one; finish() hands over the last.
template <bool HULL>
struct LaneWalk {
    const RowPath<HULL> &p;
    const GridDev &g;
    double w[3];    // the path's position (mm)
    double f[3];    // and its voxel, from -1 to n
    int i[3];
    unsigned j;     // linear index of it (wraps outside the grid)
    double c;       // mm of the path in it so far
    bool onward;    // the path has moved on along axis `dom` in every segment
    int dom;
    double sgn;

    __device__ __forceinline__ LaneWalk(const RowPath<HULL> &path, const GridDev &grid, const Rec &r)
        : p(path), g(grid), c(0.0), onward(true), dom(dominant_axis(r)), sgn((dom ? r.sn : r.cs) > 0.0 ? 1.0 : -1.0)
    {
        place(0, w);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            f[a] = voxel(a, w[a]);
            i[a] = int(f[a]);
        }
        j = unsigned(i[0]) + unsigned(g.n[0]) * (unsigned(i[1]) + unsigned(g.n[1]) * unsigned(i[2]));
    }
    __device__ __forceinline__ void place(int k, double x[3]) const { p.place(k, p.fetch(k), x[0], x[1], x[2]); }
    __device__ __forceinline__ double voxel(int a, double x) const
    {
        return fmin(fmax(floor((x - g.lo[a]) * g.inv_pitch[a]), -1.0), double(g.n[a]));
    }
    __device__ __forceinline__ double plane(int a, double x) const { return fma(x, g.pitch[a], g.lo[a]); }
    template <class Sink>
    __device__ __forceinline__ void leave(Sink &sink)
    {
        if (c > 0.0 && unsigned(i[0]) < unsigned(g.n[0]) && unsigned(i[1]) < unsigned(g.n[1]) &&
            unsigned(i[2]) < unsigned(g.n[2]))
            sink.piece(int(j), i[0], i[1], i[2], c);
        c = 0.0;
    }
    template <class Sink>
    __device__ __forceinline__ void finish(Sink &sink)
    {
        leave(sink);
    }
    template <class Sink>
    __device__ __forceinline__ void run(int k0, int k1, Sink &sink)
    {
        const unsigned stride[3] = {1u, unsigned(g.n[0]), unsigned(g.n[0]) * unsigned(g.n[1])};
        for (int k = k0; k < k1; ++k) {
            double w1[3], f1[3], d[3], at[3];
            place(k + 1, w1);
            double len2 = 0.0;
            bool far = false;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                d[a] = w1[a] - w[a];
                f1[a] = voxel(a, w1[a]);
                len2 = fma(d[a], d[a], len2);
            }
            if (k + 1 == p.K) {  // a path that ends on a plane has not crossed it
#pragma unroll
                for (int a = 0; a < 3; ++a)
                    if (d[a] > 0.0 && w1[a] == plane(a, f1[a])) f1[a] -= 1.0;
            }
            onward = onward && (dom ? d[1] : d[0]) * sgn > 0.0;
            const double len = fast_sqrt(len2);
            int e[3];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                e[a] = int(f1[a]) - i[a];
                far |= unsigned(e[a] + 1) > 2u;
                at[a] = 2.0;
                // (a crossing lies in its segment, also where the path runs along the
                // plane and its vertices' last bits cross it: there the quotient is
                // of two rounding errors)
                if (e[a] != 0)
                    at[a] = fmin(fmax((plane(a, fmax(f[a], f1[a])) - w[a]) * fast_rcp(d[a]), 0.0), 1.0);
            }
            double last = 0.0;
            if (!__any(far)) {
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    const double best = fmin(at[0], fmin(at[1], at[2]));
                    if (!(best < 1.5)) break;
                    c = fma(best - last, len, c);
                    leave(sink);
                    last = best;
                    const bool bx = at[0] == best, by = !bx && at[1] == best, bz = !bx && !by;
                    if (bx) i[0] += e[0], j += unsigned(e[0]) * stride[0], at[0] = 2.0;
                    if (by) i[1] += e[1], j += unsigned(e[1]) * stride[1], at[1] = 2.0;
                    if (bz) i[2] += e[2], j += unsigned(e[2]) * stride[2], at[2] = 2.0;
                }
            } else {
                double inv[3];
                auto next = [&](int a) {
                    const double to = plane(a, double(i[a]) + (e[a] > 0 ? 1.0 : 0.0));
                    at[a] = e[a] == 0 ? 2.0 : fmin(fmax((to - w[a]) * inv[a], last), 1.0);
                };
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    inv[a] = fast_rcp(d[a]);
                    next(a);
                }
                for (;;) {
                    const double best = fmin(at[0], fmin(at[1], at[2]));
                    if (!(best < 1.5)) break;
                    c = fma(best - last, len, c);
                    leave(sink);
                    last = best;
                    const bool bx = at[0] == best, by = !bx && at[1] == best, bz = !bx && !by;
                    auto step = [&](int a) {
                        const int s = e[a] > 0 ? 1 : -1;
                        i[a] += s;
                        j += unsigned(s) * stride[a];
                        e[a] -= s;
                        next(a);
                    };
                    if (bx) step(0);
                    if (by) step(1);
                    if (bz) step(2);
                }
            }
            c = fma(1.0 - last, len, c);
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                w[a] = w1[a];
                f[a] = f1[a];
            }
        }
    }
};

// Pointers that name their address space: a probe or a store through a generic
// one would be a flat access, which waits for LDS and HBM both.
template <typename V>
using LdsPtr = __attribute__((address_space(3))) V *;
template <typename V>
using HbmPtr = __attribute__((address_space(1))) V *;

constexpr int kWG = 256;  // lanes of a workgroup with a row each

// Re-entry tracker.  A voxel can be visited again only while the path stays in
// one slab of the dominant in-plane axis (the path is monotone along it), and
// only after the index along one of the two other axes has reversed direction
// inside that slab, or where the path left the grid and came back.  Until then
// every piece is a first visit; afterwards pieces are looked up among the slab's
// last R, which each lane keeps in LDS (a register window has to be shifted for
// every piece, and is read by one row in thousands).  If they are not all of the
// slab the proton is flagged (PCT_DEV_REENTRY).
struct Reentry {
    static constexpr int R = 8;
    struct Lds {
        int j[R][kWG];
        double c[R][kWG];
    };
    LdsPtr<int> rj;
    LdsPtr<double> rc;
    int dom;
    int k = 0;                        // pieces of the slab before this one
    int pa = -1, pb = 0, pz = 0;      // the piece before: slab, the two other indices
    int sb = 0, sz = 0;               // last steps along them inside the slab
    bool rev = false, unsafe = false;

    __device__ __forceinline__ Reentry(Lds &lds, const Rec &r)
        : rj((LdsPtr<int>)&lds.j[0][threadIdx.x]), rc((LdsPtr<double>)&lds.c[0][threadIdx.x]), dom(dominant_axis(r))
    {
    }

    // Registers piece (j, c); returns the sum of the chords of the row's earlier
    // pieces in the same voxel (0 on a first visit) and sets `first`.
    __device__ __forceinline__ double visit(int j, int ix, int iy, int iz, double c, bool &first)
    {
        const int a = dom ? iy : ix, b = dom ? ix : iy;
        const bool same = a == pa;
        const int db = same ? b - pb : 0, dz = same ? iz - pz : 0;
        auto back = [](int d, int s) { return d != 0 && s != 0 && (d ^ s) < 0; };
        rev = same && (rev || (db | dz) == 0 || back(db, sb) || back(dz, sz));
        sb = db != 0 || !same ? db : sb;
        sz = dz != 0 || !same ? dz : sz;
        k = same ? k + 1 : 0;
        pa = a;
        pb = b;
        pz = iz;
        double before = 0.0;
        first = true;
        if (rev) {
            unsafe |= k > R;
            for (int q = max(k - R, 0); q < k; ++q) {
                if (rj[(q % R) * kWG] != j) continue;
                before += rc[(q % R) * kWG];
                first = false;
            }
        }
        rj[(k % R) * kWG] = j;
        rc[(k % R) * kWG] = c;
        return before;
    }
};

}  // namespace pct
