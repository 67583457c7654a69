// Row walk of one wave: the path of one proton as a list of records in LDS,
// then its pieces.
//
// First the wave takes the polyline's segments, one per lane: a lane forms its
// segment's end vertex and the voxel that vertex is in, so the number of grid
// planes the segment crosses is the distance of two voxel indices, and a prefix
// sum over the lanes gives every crossing its place in the row's list.  A
// crossing's record holds its segment, its distance from the segment's start,
// and the voxel the path is in after it.  Then the wave takes the records, one
// per lane: piece i runs from record i to record i + 1, so consecutive pieces in
// a voxel are merged by construction, its length is the sum of what the path
// covers of each segment, and its neighbours in the list tell whether the voxel
// or the slab was met before.
//
// Against a lane walking its own share of the path from plane to plane, no lane
// waits for another's crossings: both halves are straight code with all lanes
// busy (220 segments and 290 pieces per row on the head grid), where the
// walking lanes branched between three axes and the wave paid for each branch.
#pragma once

#include "pct_path.hpp"

namespace pct {

// A crossing: its distance from the start of its segment (mm), and the voxel
// after it (ix + iy 2^xy_shift, iz; indices run from -1 to n, one past the grid
// each way).
struct RowRec {
    double s;
    int xy, z;
};
static_assert(sizeof(RowRec) + sizeof(unsigned short) == kRecBytes, "record_bytes reckons with it");

// The two fields of a packed in-plane index.
__device__ __forceinline__ int pack_xy(const GridDev &g, int ix, int iy) { return ix + iy * (1 << g.xy_shift); }
__device__ __forceinline__ int rec_ix(const GridDev &g, int xy) { return __builtin_amdgcn_sbfe(xy, 0, g.xy_shift); }
__device__ __forceinline__ int rec_iy(const GridDev &g, int xy) { return (xy - rec_ix(g, xy)) >> g.xy_shift; }

// 1 / d to the last bit or two: hardware estimate and two Newton steps.
__device__ __forceinline__ double fast_rcp(double d)
{
    double r = __builtin_amdgcn_rcp(d);
    r = fma(fma(-d, r, 1.0), r, r);
    return fma(fma(-d, r, 1.0), r, r);
}

// sqrt(x) to the last bit or two; 0 below the least normal number.
__device__ __forceinline__ double fast_sqrt(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    double s = x * y, h = 0.5 * y;
    const double e = fma(-h, s, 0.5);
    s = fma(s, e, s);
    h = fma(h, e, h);
    s = fma(fma(-s, s, x), h, s);
    return x > 0x1p-1000 ? s : 0.0;
}

// ---- lanes of a wave -------------------------------------------------------
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ int dpp(int v)  // 0 from beyond the wave or an unselected row
{
    return __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xf, false);
}
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ double dpp(double v)
{
    return __hiloint2double(dpp<CTRL, ROWS>(__double2hiint(v)), dpp<CTRL, ROWS>(__double2loint(v)));
}
constexpr int kRowShr = 0x110, kWaveShr = 0x138, kBcast15 = 0x142, kBcast31 = 0x143;

// Inclusive prefix sum over the wave.
template <typename V>
__device__ __forceinline__ V wave_scan(V v)
{
    v += dpp<kRowShr + 1>(v);
    v += dpp<kRowShr + 2>(v);
    v += dpp<kRowShr + 4>(v);
    v += dpp<kRowShr + 8>(v);
    v += dpp<kBcast15, 0xa>(v);
    v += dpp<kBcast31, 0xc>(v);
    return v;
}
__device__ __forceinline__ int lane_value(int v, int lane) { return __builtin_amdgcn_readlane(v, lane); }
__device__ __forceinline__ double lane_value(double v, int lane)
{
    return __hiloint2double(lane_value(__double2hiint(v), lane), lane_value(__double2loint(v), lane));
}
template <typename V>
__device__ __forceinline__ V wave_sum(V v)
{
    return lane_value(wave_scan(v), kWave - 1);
}
// v of the lane before, `first` in lane 0
__device__ __forceinline__ int lane_before(int v, int first)
{
    return __builtin_amdgcn_update_dpp(first, v, kWaveShr, 0xf, 0xf, false);
}
__device__ __forceinline__ double lane_before(double v, double first)
{
    return __hiloint2double(lane_before(__double2hiint(v), __double2hiint(first)),
                            lane_before(__double2loint(v), __double2loint(first)));
}

// ---- the row -----------------------------------------------------------------
// Dominant in-plane axis of a row (0: x, 1: y).
__device__ __forceinline__ int dominant_axis(const Rec &r) { return fabs(r.cs) >= fabs(r.sn) ? 0 : 1; }

// Index along axis a of the voxel that holds w (mm), clamped to one voxel beyond
// the grid.  (A point within rounding of a plane may be put on
// either side: its crossing then falls on the segment's end.)
__device__ __forceinline__ int voxel_index(double w, const GridDev &g, int a)
{
    return int(fmin(fmax(floor((w - g.lo[a]) * g.inv_pitch[a]), -1.0), double(g.n[a])));
}
__device__ __forceinline__ double plane_at(int i, const GridDev &g, int a)
{
    return fma(double(i), g.pitch[a], g.lo[a]);
}

// What one wave needs of its row (the same in every lane).  With a hull the
// straight parts outside it are cut into steps too, so that no segment crosses
// a long run of planes.
template <bool HULL>
struct RowPath {
    const PathSrc &src;
    const GridDev &g;
    Rec r;
    PathState ps;
    int K;          // segments
    int k_in, k_out;  // hull: segments before it and after it
    __device__ __forceinline__ RowPath(const PathSrc &src_, const GridDev &g_, const Rec &r_)
        : src(src_), g(g_), r(r_), ps(path_prepare<HULL>(r_, src_)), K(src_.K), k_in(0), k_out(0)
    {
        if constexpr (HULL) {
            if (!ps.miss) {
                // (a length that is a whole number of steps up to rounding is cut
                // into that many: one cut more would fall on the hull point)
                auto steps = [&](double length) {
                    return length > 0.0 ? max(1, int(ceil(length * src.inv_step - 0x1p-30))) : 0;
                };
                k_in = steps(ps.uh_in - src.u_in);
                k_out = steps(src.u_out - ps.uh_out);
                K = k_in + ps.kh + k_out;
            }
        }
    }
    // Row of the shared table, or the vertex itself on a hull path.
    struct Vertex {
        double c[5];
    };
    __device__ __forceinline__ Vertex fetch(int k) const
    {
        Vertex v{};
        if constexpr (!HULL) {
            const double *__restrict__ row = src.tab + k * kRowDoubles;
#pragma unroll
            for (int q = 0; q < 5; ++q) v.c[q] = row[q];
        }
        return v;
    }
    // vertex k (mm; from the grid's corner it would be twice as large, and as
    // coarse)
    __device__ __forceinline__ void place(int k, const Vertex &c, double &x, double &y, double &z) const
    {
        double u, t, v;
        if constexpr (HULL) {
            if (ps.miss) {
                const double w = double(k) / double(K);
                u = k == K ? src.u_out : src.u_in + w * (src.u_out - src.u_in);
                t = k == K ? r.t_out : r.t_in + w * (r.t_out - r.t_in);
                v = k == K ? r.v_out : r.v_in + w * (r.v_out - r.v_in);
            } else if (k < k_in) {
                u = src.u_in + double(k) * src.step;
                t = r.t_in + r.th_in * (u - src.u_in);
                v = r.v_in + r.ph_in * (u - src.u_in);
            } else if (k > K - k_out) {
                u = src.u_out - double(K - k) * src.step;
                t = r.t_out - r.th_out * (src.u_out - u);
                v = r.v_out - r.ph_out * (src.u_out - u);
            } else {
                hull_point(r, src, ps, k - k_in, u, t, v);
            }
        } else {
            t = c.c[0] * r.t_in + c.c[1] * r.th_in + c.c[2] * r.t_out + c.c[3] * r.th_out;
            v = c.c[0] * r.v_in + c.c[1] * r.ph_in + c.c[2] * r.v_out + c.c[3] * r.ph_out;
            u = c.c[4];
        }
        x = u * r.cs - t * r.sn;
        y = u * r.sn + t * r.cs;
        z = v;
    }
};

// Window of a row's record list in LDS: records [lo - kRecPad, lo + span +
// kLookAhead] of the list, for the pieces [lo, lo + span) (span is a multiple of
// the wave).
struct RecWindow {
    RowRec *rec;
    unsigned short *seg;  // segment of each record
    double *len;          // length of every segment of the row
    int span;
    int lo = 0, n = 0;    // n: pieces of the row
    // In the workgroup's LDS: lengths of up to `segments` segments, records, segments.
    __device__ __forceinline__ RecWindow(double *lds, int segments, int span_)
        : rec(reinterpret_cast<RowRec *>(lds + ((segments + 1) & ~1))),
          seg(reinterpret_cast<unsigned short *>(rec + span_ + kRecPad + 1 + kLookAhead)), len(lds), span(span_)
    {
    }
    __device__ __forceinline__ int slot(int i) const { return i - lo + kRecPad; }
    __device__ __forceinline__ RowRec *at(int i) const { return rec + slot(i); }
    __device__ __forceinline__ void put(int i, int k, double s, int xy, int z) const
    {
        if (unsigned(slot(i)) > unsigned(span + kRecPad + kLookAhead)) return;
        rec[slot(i)] = RowRec{s, xy, z};
        seg[slot(i)] = static_cast<unsigned short>(k);
    }
    // path between records i and i + 1
    __device__ __forceinline__ double length(int i) const
    {
        const double s0 = at(i)->s, s1 = at(i + 1)->s;
        int k0 = seg[slot(i)];
        const int k1 = seg[slot(i + 1)];
        if (k0 == k1) return s1 - s0;
        double c = (len[k0] - s0) + s1;
        while (++k0 < k1) c += len[k0];
        return c;
    }
};

// Crossings of one segment that passes more than one plane of an axis: one
// after the other.
__device__ __forceinline__ void put_many(const RecWindow &win, const GridDev &g, int i, int k, double len,
                                         const double w0[3], const double w1[3], const int i0[3], const int i1[3])
{
    int at[3] = {i0[0], i0[1], i0[2]};
    double inv[3], f[3];  // fraction of the segment at the next plane of each axis
    auto next = [&](int a) {
        const double plane = plane_at(i1[a] > at[a] ? at[a] + 1 : at[a], g, a);
        f[a] = at[a] == i1[a] ? 2.0 : fmin(fmax((plane - w0[a]) * inv[a], 0.0), 1.0);
    };
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        inv[a] = fast_rcp(w1[a] - w0[a]);
        next(a);
    }
    double last = 0.0;
    for (;;) {
        const double best = fmin(f[0], fmin(f[1], f[2]));
        if (best > 1.0) return;
        last = fmax(last, best);
        bool done = false;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            if (!done && f[a] == best) {
                at[a] += i1[a] > at[a] ? 1 : -1;
                next(a);
                done = true;
            }
        }
        win.put(i++, k, last * len, pack_xy(g, at[0], at[1]), at[2]);
    }
}

// What the walk tells of a row besides its pieces (the same in every lane).
struct RowShape {
    bool onward = true;  // the path moves on along the dominant axis in every segment
    bool turns = false;  // its voxel index goes both ways along some axis: without, no voxel comes back
    bool cut = false;    // a voxel may have come back from before the window
};

// The records of the window, the number of pieces of the row, and its shape.  All
// lanes of the wave call it; the caller waits for the LDS writes.
template <bool HULL>
__device__ __forceinline__ int row_records(const RowPath<HULL> &p, const RecWindow &win, int dom, RowShape &shape)
{
    const GridDev &g = p.g;
    const int lane = int(threadIdx.x) & (kWave - 1);
    double cx, cy, cz;  // start of the round's first segment
    p.place(0, p.fetch(0), cx, cy, cz);
    auto ahead = p.fetch(min(lane + 1, p.K));  // of the round to come
    int jx = voxel_index(cx, g, 0), jy = voxel_index(cy, g, 1), jz = voxel_index(cz, g, 2);
    const int sx = lane_value(jx, 0), sy = lane_value(jy, 0), sz = lane_value(jz, 0);
    int n = 1;  // records before this round
    bool onward = true;
    const double sgn = (dom ? p.r.sn : p.r.cs) > 0.0 ? 1.0 : -1.0;
    if (lane == 0) win.put(0, 0, 0.0, pack_xy(g, jx, jy), jz);
    for (int k0 = 0; k0 < p.K; k0 += kWave) {
        const int k = min(k0 + lane + 1, p.K);  // the segment's end (none beyond the last: empty segments)
        double x1, y1, z1;
        p.place(k, ahead, x1, y1, z1);
        ahead = p.fetch(min(k0 + kWave + lane + 1, p.K));
        const double x0 = lane_before(x1, cx), y0 = lane_before(y1, cy), z0 = lane_before(z1, cz);
        const double dx = x1 - x0, dy = y1 - y0, dz = z1 - z0;
        int ix1 = voxel_index(x1, g, 0), iy1 = voxel_index(y1, g, 1), iz1 = voxel_index(z1, g, 2);
        if (k == p.K) {  // a path that ends on a plane has not crossed it
            ix1 -= dx > 0.0 && x1 == plane_at(ix1, g, 0) ? 1 : 0;
            iy1 -= dy > 0.0 && y1 == plane_at(iy1, g, 1) ? 1 : 0;
            iz1 -= dz > 0.0 && z1 == plane_at(iz1, g, 2) ? 1 : 0;
        }
        const bool on = k0 + lane < p.K;
        const int ix0 = lane_before(ix1, jx), iy0 = lane_before(iy1, jy), iz0 = lane_before(iz1, jz);
        if (!on) {
            ix1 = ix0;
            iy1 = iy0;
            iz1 = iz0;
        }
        const int ex = ix1 - ix0, ey = iy1 - iy0, ez = iz1 - iz0;
        const double len = fast_sqrt(fma(dx, dx, fma(dy, dy, dz * dz)));
        const int count = abs(ex) + abs(ey) + abs(ez);
        const int past = wave_scan(count);
        if (on) win.len[k0 + lane] = len;
        const int first = n + past - count;
        onward = onward && __all(!on || (dom ? dy : dx) * sgn > 0.0);
        if (__any(abs(ex) > 1 || abs(ey) > 1 || abs(ez) > 1)) {
            const double w0[3] = {x0, y0, z0}, w1[3] = {x1, y1, z1};
            const int i0[3] = {ix0, iy0, iz0}, i1[3] = {ix1, iy1, iz1};
            put_many(win, g, first, k0 + lane, len, w0, w1, i0, i1);
        } else {
            // fraction of the segment at each crossing (2: none) and their order
            auto fraction = [&](int e, int i0, double w0, double d, int a) {
                const double plane = plane_at(i0 + (e > 0 ? 1 : 0), g, a);
                return e != 0 ? fmin(fmax((plane - w0) * fast_rcp(d), 0.0), 1.0) : 2.0;
            };
            const double fx = fraction(ex, ix0, x0, dx, 0), fy = fraction(ey, iy0, y0, dy, 1),
                         fz = fraction(ez, iz0, z0, dz, 2);
            const bool xy = fx <= fy, xz = fx <= fz, yz = fy <= fz;
            const int at = pack_xy(g, ix0, iy0), ey2 = pack_xy(g, 0, ey);
            if (ex != 0)
                win.put(first + (xy ? 0 : 1) + (xz ? 0 : 1), k0 + lane, fx * len, at + ex + (xy ? 0 : ey2),
                        iz0 + (xz ? 0 : ez));
            if (ey != 0)
                win.put(first + (xy ? 1 : 0) + (yz ? 0 : 1), k0 + lane, fy * len, at + ey2 + (xy ? ex : 0),
                        iz0 + (yz ? 0 : ez));
            if (ez != 0)
                win.put(first + (xz ? 1 : 0) + (yz ? 1 : 0), k0 + lane, fz * len,
                        at + (xz ? ex : 0) + (yz ? ey2 : 0), iz0 + ez);
        }
        n += lane_value(past, kWave - 1);
        cx = lane_value(x1, kWave - 1);
        cy = lane_value(y1, kWave - 1);
        cz = lane_value(z1, kWave - 1);
        jx = lane_value(ix1, kWave - 1);
        jy = lane_value(iy1, kWave - 1);
        jz = lane_value(iz1, kWave - 1);
    }
    shape.onward = onward;
    // a crossing is a step of one index: more of them than the ends are apart
    shape.turns = n - 1 != abs(jx - sx) + abs(jy - sy) + abs(jz - sz);
    // the list's end
    __syncthreads();
    if (lane <= kLookAhead) win.put(n + lane, p.K - 1, win.len[p.K - 1], pack_xy(g, -2, -2), -2);
    return n;
}

// One piece of a row, as the consumer of row_pieces sees it.
struct RowPiece {
    int ix, iy, iz;
    double c;     // length (mm), already rounded to the chord format
    bool real;    // of positive length, inside the grid
    int more;     // records of the slab after this one, up to 3
    bool first;   // the row has not met the voxel before
    double before;  // length of the row's earlier pieces in the voxel
    int slab, k;  // slab of the dominant axis, and records of it before this one
};

// Calls use(piece) for every record of the row, 64 at a time in path order (all
// lanes of the wave take part; lanes beyond the list get a piece that is not
// real and has k < 0).  `have`: the window holds the row already.
//
// A voxel can be met again inside its slab only, and not before two pieces on,
// where the path moves on along the dominant axis: a piece looks back over its
// slab.  A row of several windows keeps the slab it is in from one to the next;
// where a slab does not fit a window, a piece of a path that turns somewhere and
// would look back further raises shape.cut.  A path that turns back along that axis may meet any voxel again, and its pieces
// look back over the window.
template <bool HULL, int CHORD, class Use>
__device__ __forceinline__ void row_pieces(const RowPath<HULL> &p, RecWindow &win, int dom, bool &have,
                                           RowShape &shape, Use &&use)
{
    const GridDev &g = p.g;
    const int lane = int(threadIdx.x) & (kWave - 1);
    int run = 0, slab_before = INT_MIN;  // of the slab the round before ended in
    int n = 0;
    for (int lo = 0, from = 0; from == 0 || from < n;) {  // window, and the first piece that it hands over
        if (!(have && from == 0)) {
            win.lo = lo;
            __syncthreads();
            n = row_records<HULL>(p, win, dom, shape);
            __syncthreads();
            win.n = n;
        }
        n = win.n;
        const int hi = min(n, lo + win.span);
        for (int g0 = from; g0 < hi; g0 += kWave) {
            const int i = g0 + lane;
            const bool on = i < hi;
            const RowRec a = *win.at(on ? i : hi);
            const int b_xy = win.at(on ? i + 1 : hi)->xy;
            const double length = on ? win.length(i) : 0.0;
            RowPiece q;
            q.ix = rec_ix(g, a.xy);
            q.iy = rec_iy(g, a.xy);
            q.iz = a.z;
            q.c = round_chord<CHORD>(length);
            q.real = length > 0.0 && unsigned(q.ix) < unsigned(g.n[0]) && unsigned(q.iy) < unsigned(g.n[1]) &&
                     unsigned(q.iz) < unsigned(g.n[2]);
            q.slab = dom ? q.iy : q.ix;
            auto slab_of = [&](int xy) { return dom ? rec_iy(g, xy) : rec_ix(g, xy); };
            q.more = slab_of(b_xy) != q.slab ? 0
                     : slab_of(win.at(min(i + 2, hi + kLookAhead))->xy) != q.slab ? 1
                     : slab_of(win.at(min(i + 3, hi + kLookAhead))->xy) != q.slab ? 2 : 3;
            const unsigned long long starts = __ballot(q.slab != lane_before(q.slab, slab_before));
            const unsigned long long below = starts & (~0ull >> (kWave - 1 - lane));
            q.k = !on ? -1 : below != 0ull ? lane - (kWave - 1 - __clzll(below)) : run + lane;
            q.first = true;
            q.before = 0.0;
            if (shape.turns) {
                int back = !q.real ? 0 : shape.onward ? q.k : i;
                if (lo > 0) {
                    const int stored = i - lo + min(lo, kRecPad);
                    shape.cut |= __any(back > stored);
                    back = min(back, stored);
                }
                for (int d = 2; d <= back; ++d) {
                    const RowRec *e = win.at(i - d);
                    if (e->xy != a.xy || e->z != a.z) continue;
                    const double c = win.length(i - d);
                    if (c > 0.0) {
                        q.first = false;
                        q.before += round_chord<CHORD>(c);
                    }
                }
            }
            use(q);
            run = starts != 0ull ? kWave - (kWave - 1 - __clzll(starts)) : run + kWave;
            slab_before = lane_value(q.slab, kWave - 1);
        }
        const int slab = (run + kWave - 1) & -kWave;
        from = hi;
        lo = hi - (!shape.onward ? 0 : slab < win.span ? slab : (win.span / 2) & -kWave);
    }
    have = n <= win.span;
}

}  // namespace pct
