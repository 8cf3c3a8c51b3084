// The interface kernel of rectangular hexahedra (gfx950, wave64, FP64): the same construction as
// k_surface (vertex values, isovalue, isoface, swept faces; Section 3.2) on cells whose edges run
// along the coordinate axes, written in the cell's own coordinates (0 to 1 along each edge).
//
// Two lanes per interface cell.  Lane 0 owns the three faces that meet at the cell's first vertex,
// lane 1 the three at the opposite vertex, each in local coordinates that start at its own vertex
// (lane 1's are 1 - x), so both run the same code with their faces at local coordinate 0.  There a
// face is the unit square of two of the coordinates, a cut point is one edge parameter
// t = (iso - a_i) / (a_j - a_i), and the sub-volume about the isoface's apex o is the sum over the
// six faces of o's distance to the face times the face's wet area: no cross products in 3D, no
// volume term of the isoface itself.  Physical lengths enter through the squared edge lengths alone.
//
// What bounds it: on small meshes the chain of one wave (about 3000 VALU instructions, half of them FP64
// arithmetic at four cycles each or eight when dependent, and five dependent loads of 1 us each); on
// large ones also the vector caches (the stencils' 96 bytes of each vertex).  Against the general
// kernel's eight lanes per cell (about 4900 VALU instructions per wave of 8 cells): 13.5 us instead of
// 26.0 for 72 interface cells of a slab, 16 instead of 27.9 for 1136, 25.3 instead of 97.9 for the 46.5k of
// the 256x128x128 box.  Rounding: of one step of 90 graded boxes against 80-bit arithmetic, the largest error
// of a box is on average 0.77 of the general kernel's and its root mean square 0.81 (the reciprocals and
// roots below are good to a unit in the last place, but there are fewer operations).
// Two lanes rather than one or eight: one lane would halve the waves, which at 45k cells are already
// only 1.4 per SIMD, and eight would spend most of each wave on the same scalar steps of the search.
#include "device_common.h"

namespace isoadv {
namespace {

__device__ __forceinline__ double swap1(double v) { return dpp_move<kDppSwap1>(v); }  // the other lane's value

// Reciprocal to about one unit in the last place: the hardware's estimate and two Newton steps.  A
// difference too small for its reciprocal to be finite counts as zero, whose reciprocal is taken as 0.
constexpr double kTiny = 1e-290;
__device__ __forceinline__ double recip(double d) {
    double r = __builtin_amdgcn_rcp(d);
    r = fma(fma(-d, r, 1.0), r, r);
    r = fma(fma(-d, r, 1.0), r, r);
    return fabs(d) > kTiny ? r : 0.0;
}

// a * b + c in a register of its own (the compiler's fused form overwrites c, after copying it).
__device__ __forceinline__ double fma3(double a, double b, double c) {
    double d;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
    return d;
}

// a * b clamped to [0, 1] (the clamp is free on the multiplication).
__device__ __forceinline__ double mul01(double a, double b) {
    double d;
    asm("v_mul_f64 %0, %1, %2 clamp" : "=v"(d) : "v"(a), "v"(b));
    return d;
}
// Smaller and larger of two numbers, one instruction each (the library forms first quiet operands
// whose origin they cannot see).
__device__ __forceinline__ double min2(double a, double b) {
    double d;
    asm("v_min_f64 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b));
    return d;
}
__device__ __forceinline__ double max2(double a, double b) {
    double d;
    asm("v_max_f64 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b));
    return d;
}

// c ? a : b on values held in registers.
__device__ __forceinline__ double pick(bool c, double a, double b) {
    asm("" : "+v"(a), "+v"(b));
    return c ? a : b;
}

// Square root and its reciprocal (Goldschmidt's iteration from the hardware's estimate, then one
// correction of the root); x below kTiny counts as kTiny.
struct Root {
    double s, r;
};
__device__ __forceinline__ Root root(double x) {
    x = max2(x, kTiny);
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    const double e = fma(-h, g, 0.5);
    g = fma(g, e, g);
    h = fma(h, e, h);
    g = fma(fma(-g, g, x), h, g);
    return {g, h + h};
}

// Local vertex i + 2j + 4k sits at local coordinates (i, j, k).  Edges by their ends; vertex 7 is
// on none of the lane's faces.
constexpr int kBoxEdge[9][2] = {{0, 1}, {0, 2}, {0, 4}, {2, 6}, {4, 6}, {4, 5}, {1, 5}, {1, 3}, {2, 3}};
// Face f lies at local coordinate f = 0, its square in coordinates p = f + 1 and q = f + 2 (mod 3):
// corners c0 (0,0), c1 (1,0), c2 (1,1), c3 (0,1), and the edges E0 c0-c1, E1 c1-c2, E2 c3-c2, E3
// c0-c3, their parameters running along +p or +q.
constexpr int kBoxCorner[3][4] = {{0, 2, 6, 4}, {0, 4, 5, 1}, {0, 1, 3, 2}};
constexpr int kBoxFaceEdge[3][4] = {{1, 3, 4, 2}, {2, 5, 6, 0}, {0, 7, 8, 1}};
// Canonical vertex at cell coordinates (bits i, j, k), one per nibble.
constexpr uint32_t kBoxCanon = 0x67542310u;
// Canonical face at cell coordinate f = 0 (lane 0) and f = 1 (lane 1).
constexpr int kBoxFace[2][3] = {{5, 2, 0}, {3, 4, 1}};

// An isoface edge on a face's square, from the exit to the entry cut of the wet part's walk: twice its
// midpoint and the vector along it.
struct Edge2 {
    double mp, mq, dp, dq;
};
__device__ __forceinline__ Edge2 operator-(Edge2 a, Edge2 b) { return {a.mp - b.mp, a.mq - b.mq, a.dp - b.dp, a.dq - b.dq}; }
__device__ __forceinline__ double cross2(const Edge2 &a, const Edge2 &b) { return fma(a.mp, b.dq, -(a.mq * b.dp)); }

struct Cell {
    double a[8];    // vertex values, local order
    double inv[9];  // reciprocal differences along the edges; an edge of equal values counts as falling
                    // without end, so that its wet part is all of it or nothing
    double up[9];   // 1 where the value rises along the edge, else 0
    double gm[3];   // squared edge lengths over the largest
};

// Where the isovalue x cuts the edges, as parameters clamped to [0, 1].
__device__ __forceinline__ void cut_points(const Cell &c, double x, double *t) {
#pragma unroll
    for (int e = 0; e < 9; ++e) t[e] = mul01(x - c.a[kBoxEdge[e][0]], c.inv[e]);
}

// A face's isoface edge from its four edges' values: y whose magnitude is the wet part of each edge, s
// the cut points and k ones (both zero on edges that are not cut).  The wet parts, walked around the
// face, and the isoface edge close; so its vector is the difference of the opposite edges' wet parts,
// and its ends are the two cut points.  On a saddle (all four edges cut) this is the sum of its two
// edges.
__device__ __forceinline__ Edge2 face_edge(int f, const double *y, const double *s, const double *k) {
    const int *e = kBoxFaceEdge[f];
    return {s[e[0]] + k[e[1]] + s[e[2]], s[e[1]] + k[e[2]] + s[e[3]], fabs(y[e[2]]) - fabs(y[e[0]]), fabs(y[e[3]]) - fabs(y[e[1]])};
}

// The second isoface edge of saddle face f at isovalue x (around corner c3 when c0 is wet, around c2
// otherwise), and its rate of change.
__device__ __forceinline__ void second_edge(const Cell &c, int f, bool wet0, double x, Edge2 &e, Edge2 &r) {
    const int *n = kBoxFaceEdge[f];
    const double i2 = c.inv[n[2]], t2 = mul01(x - c.a[kBoxEdge[n[2]][0]], i2);
    // both sides formed, then one picked: a pick between the array elements themselves would put the
    // arrays into memory
    const double i1 = pick(wet0, c.inv[n[3]], c.inv[n[1]]);
    const double t1 = pick(wet0, mul01(x - c.a[kBoxEdge[n[3]][0]], c.inv[n[3]]), mul01(x - c.a[kBoxEdge[n[1]][0]], c.inv[n[1]]));
    e = wet0 ? Edge2{t2, 1.0 + t1, -t2, t1 - 1.0} : Edge2{1.0 + t2, t1 + 1.0, t2 - 1.0, 1.0 - t1};
    r = wet0 ? Edge2{i2, i1, -i2, i1} : Edge2{i2, i1, i2, -i1};
}

// Sums over isoface edges in the lane's local coordinates: length, and length times twice the midpoint.
// Of each face the edge has no component along the face's own coordinate.
struct Perimeter {
    double l, m[3];
};
__device__ __forceinline__ double edge_length2(const Cell &c, int f, const Edge2 &e) {
    return fma(c.gm[(f + 1) % 3] * e.dp, e.dp, (c.gm[(f + 2) % 3] * e.dq) * e.dq);
}
__device__ __forceinline__ Perimeter perimeter(const Cell &c, const Edge2 *e) {
    double l[3];
#pragma unroll
    for (int f = 0; f < 3; ++f) l[f] = root(edge_length2(c, f, e[f])).s;
    return {l[0] + l[1] + l[2],
            {fma(l[2], e[2].mp, l[1] * e[1].mq), fma(l[0], e[0].mp, l[2] * e[2].mq), fma(l[1], e[1].mp, l[0] * e[0].mq)}};
}
__device__ __forceinline__ void add_edge(const Cell &c, int f, const Edge2 &e, Perimeter &s) {
    const double l = root(edge_length2(c, f, e)).s;
    s.l += l;
    s.m[(f + 1) % 3] = fma(l, e.mp, s.m[(f + 1) % 3]);
    s.m[(f + 2) % 3] = fma(l, e.mq, s.m[(f + 2) % 3]);
}

// Both lanes' sums, in the lane's coordinates (the other lane's midpoints mirrored), as twice the
// perimeter centroid.
__device__ __forceinline__ void apex(const Perimeter &s, double *o2) {
    const double l = s.l + swap1(s.l);
    const double il = recip(l);
#pragma unroll
    for (int i = 0; i < 3; ++i) o2[i] = il * (s.m[i] + swap1(fma(2.0, s.l, -s.m[i])));
}

// Which edges the wet pattern w cuts, and whether a face is a saddle.
__device__ __forceinline__ bool cut_edge(const bool *w, int e) { return w[kBoxEdge[e][0]] != w[kBoxEdge[e][1]]; }
__device__ __forceinline__ bool saddle_face(const bool *w, int f) {
    return cut_edge(w, kBoxFaceEdge[f][0]) && cut_edge(w, kBoxFaceEdge[f][1]) && cut_edge(w, kBoxFaceEdge[f][2]);
}

// Twelve times the wet share of the cell at isovalue x, a vertex wet iff its value exceeds x: over the
// faces, twice the apex's distance times twice the wet area (the wet parts of the edges away from c0,
// and the isoface edge's own term).
__device__ __forceinline__ double share12(const Cell &c, double x) {
    bool w[8];
#pragma unroll
    for (int i = 0; i < 7; ++i) w[i] = c.a[i] > x;
    double t[9], y[9], s[9], k[9];
    cut_points(c, x, t);
#pragma unroll
    for (int e = 0; e < 9; ++e) {
        const bool cut = cut_edge(w, e);
        y[e] = c.up[e] - t[e];
        s[e] = cut ? t[e] : 0.0;
        k[e] = cut ? 1.0 : 0.0;
    }
    Edge2 e[3];
    double area[3];
    bool sad[3];
#pragma unroll
    for (int f = 0; f < 3; ++f) {
        e[f] = face_edge(f, y, s, k);
        area[f] = fma(0.5, cross2(e[f], e[f]), fabs(y[kBoxFaceEdge[f][1]]) + fabs(y[kBoxFaceEdge[f][2]]));
        sad[f] = saddle_face(w, f);
    }
    Perimeter sum{0.0, {0.0, 0.0, 0.0}};
    if (sad[0] || sad[1] || sad[2]) {
#pragma unroll
        for (int f = 0; f < 3; ++f)
            if (sad[f]) {
                Edge2 e2, r2;
                second_edge(c, f, w[0], x, e2, r2);
                const Edge2 e1 = e[f] - e2;
                area[f] = fma(0.5, cross2(e1, e1) + cross2(e2, e2) - cross2(e[f], e[f]), area[f]);
                e[f] = e1;
                add_edge(c, f, e2, sum);
            }
    }
    const Perimeter first = perimeter(c, e);
    sum.l += first.l;
#pragma unroll
    for (int i = 0; i < 3; ++i) sum.m[i] += first.m[i];
    double o2[3];
    apex(sum, o2);
    const double v = fma(o2[2], area[2], fma(o2[1], area[1], o2[0] * area[0]));
    return v + swap1(v);
}

// Swept share of a rectangular face whose corners' distances from the isoface run from e0 to e0 + m + M
// (m <= M the spans along its two sides): the mean over the step of the share the plane has passed,
// moving by ud over the step (iud its reciprocal).  The share at z = distance moved - e0 is
// z^2/(2mM) up to m, (z - m/2)/M up to M, 1 - (m + M - z)^2/(2mM) up to m + M; each piece is
// integrated exactly over its part of the step, in a form whose terms are all of one sign.
__device__ __forceinline__ double rect_sweep(double e0, double m, double M, double ud, double iud) {
    const double rm = recip(m), rM = recip(M);
    const double e1 = e0 + m, e2 = e0 + M, e3 = e2 + m;
    // times of the pieces' ends as fractions of the step
    const double t0 = mul01(e0, iud), t1 = mul01(e1, iud), t2 = mul01(e2, iud), t3 = mul01(e3, iud);
    // the corner pieces in units of m, the middle one in units of M
    const double z0 = mul01(fma(ud, t0, -e0), rm), z1 = mul01(fma(ud, t1, -e0), rm);
    const double w2 = mul01(fma(-ud, t2, e3), rm), w3 = mul01(fma(-ud, t3, e3), rm);
    const double y = fma(ud, t1 + t2, -(e0 + e1));
    const double c = (m * rM) * (1.0 / 6.0);
    const double q1 = fma(z0, z0, z1 * (z0 + z1)), q3 = fma(w3, w3, w2 * (w2 + w3));
    double I = ud > 0.0 ? 1.0 - t3 : t3;
    I = fma(fabs(t1 - t0), c * q1, I);
    I = fma(fabs(t2 - t1), (0.5 * y) * rM, I);
    return fma(fabs(t3 - t2), fma(-c, q3, 1.0), I);
}

// Inverse-distance values of the vertices of kV point classes k, in stencil order, all loads of one kind in
// flight together.
template <int kN, int kV>
__device__ __forceinline__ void gather(const DevMesh &m, const double *x, const int32_t *k, double *g) {
    int32_t c[kV][kN];
    double w[kV][kN], a[kV][kN];
#pragma unroll
    for (int v = 0; v < kV; ++v) {
        const int4 *cp = reinterpret_cast<const int4 *>(m.sten_cell + (size_t)kN * k[v]);
        const double2 *wp = reinterpret_cast<const double2 *>(m.sten_w + (size_t)kN * k[v]);
#pragma unroll
        for (int j = 0; j < kN; j += 4) {
            const int4 q = cp[j / 4];
            c[v][j] = q.x; c[v][j + 1] = q.y; c[v][j + 2] = q.z; c[v][j + 3] = q.w;
        }
#pragma unroll
        for (int j = 0; j < kN; j += 2) {
            const double2 q = wp[j / 2];
            w[v][j] = q.x; w[v][j + 1] = q.y;
        }
    }
#pragma unroll
    for (int v = 0; v < kV; ++v)
#pragma unroll
        for (int j = 0; j < kN; ++j) a[v][j] = x[c[v][j]];
#pragma unroll
    for (int v = 0; v < kV; ++v) {
        g[v] = fma(w[v][0], a[v][0], 0.0);
#pragma unroll
        for (int j = 1; j < kN; ++j) g[v] = fma(w[v][j], a[v][j], g[v]);
    }
}

// The weighted sum of two vertices' velocities (components along the coordinate axes ax): the stencils of both
// first, then four cells of each at a time with all their components in flight.  Cell by cell the loads waited
// for each other; with its own registers (one wave per SIMD) the kernel went from 29.5 to 21.2 us on an outer
// iteration's 75x37x41 box and from 45.5 to 34.0 on 200x96x96, with two waves (spilled) 22.8 and 39.4.
template <int kN>
__device__ __forceinline__ void gather_velocity(const SurfArgs &A, const int (&ax)[3], const int32_t (&k)[2],
                                                const double (&w)[2], double (&us)[3]) {
    const size_t nc = A.m.n_cells;
    const double *U[3], *U1[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        U[i] = A.U + ax[i] * nc;
        U1[i] = A.U1 + ax[i] * nc;
    }
    int32_t c[2][kN];
    double sw[2][kN], uv[2][3];
#pragma unroll
    for (int v = 0; v < 2; ++v) {
        const int4 *cp = reinterpret_cast<const int4 *>(A.m.sten_cell + (size_t)kN * k[v]);
        const double2 *wp = reinterpret_cast<const double2 *>(A.m.sten_w + (size_t)kN * k[v]);
#pragma unroll
        for (int j = 0; j < kN; j += 4) {
            const int4 q = cp[j / 4];
            c[v][j] = q.x; c[v][j + 1] = q.y; c[v][j + 2] = q.z; c[v][j + 3] = q.w;
        }
#pragma unroll
        for (int j = 0; j < kN; j += 2) {
            const double2 q = wp[j / 2];
            sw[v][j] = q.x; sw[v][j + 1] = q.y;
        }
#pragma unroll
        for (int i = 0; i < 3; ++i) uv[v][i] = 0.0;
    }
#pragma unroll
    for (int j0 = 0; j0 < kN; j0 += 4) {
        double u[2][4][3];
#pragma unroll
        for (int v = 0; v < 2; ++v)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int i = 0; i < 3; ++i) u[v][j][i] = U[i][c[v][j0 + j]];
        if (A.U1) {
            double u1[2][4][3];
#pragma unroll
            for (int v = 0; v < 2; ++v)
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int i = 0; i < 3; ++i) u1[v][j][i] = U1[i][c[v][j0 + j]];
#pragma unroll
            for (int v = 0; v < 2; ++v)
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int i = 0; i < 3; ++i) u[v][j][i] = 0.5 * (u[v][j][i] + u1[v][j][i]);
        }
#pragma unroll
        for (int v = 0; v < 2; ++v)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int i = 0; i < 3; ++i) uv[v][i] = fma(sw[v][j0 + j], u[v][j][i], uv[v][i]);
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) us[i] = fma(w[1], uv[1][i], w[0] * uv[0][i]);
}

// Work-groups of one wave: the list's waves then spread evenly over the CUs (1136 interface cells of a slab
// 16.1 us against 18.6 with 256 threads, 46.5k of a box 25.3 against 26.1, interpolated velocities on 4147 cells
// of a box 16.1 against 20.4).
constexpr int kBlock = 64, kGroups = kBlock / 2;  // threads and interface cells of a work-group

// kInterp: U_S by cell-point interpolation (us_mode 1) instead of U_P.
template <bool kInterp>
__global__ void __launch_bounds__(kBlock, kInterp ? 1 : 2) k_surface_box(SurfArgs A) {
    const DevMesh &m = A.m;
    const int r = threadIdx.x & 1;
    const int n = min(A.counters[kCntSurf], A.cap);
    const size_t nc = m.n_cells;
    int rounds_max = 0, flat = 0, nonconv = 0;
    for (int idx = (blockIdx.x * kBlock + threadIdx.x) / 2; idx < n; idx += gridDim.x * kGroups) {
        const int c = A.list[idx];
        const int32_t flags = m.cflags[c];
        if (m.box == 2 && !(flags & kCellBox)) continue;  // k_surface or k_surface_big takes it
        const double aP = A.alpha[c];
        // this lane's vertices: its own and the three joined to it by an edge; the other lane has
        // the rest
        Cell cell;
        {
            double g[4];
            int32_t k[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int b = (v == 0 ? 0 : 1 << (v - 1)) ^ (r ? 7 : 0);
                k[v] = m.cpt[8 * (size_t)c + ((kBoxCanon >> (4 * b)) & 7u)];
            }
            if (m.sten_n == 4) gather<4, 4>(m, A.alpha, k, g);
            else gather<8, 4>(m, A.alpha, k, g);
            if (A.tr.vert_alpha) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int b = (v == 0 ? 0 : 1 << (v - 1)) ^ (r ? 7 : 0);
                    A.tr.vert_alpha[8 * (size_t)c + ((kBoxCanon >> (4 * b)) & 7u)] = g[v];
                }
            }
            cell.a[0] = g[0];
            cell.a[1] = g[1];
            cell.a[2] = g[2];
            cell.a[4] = g[3];
            cell.a[7] = swap1(g[0]);
            cell.a[6] = swap1(g[1]);
            cell.a[5] = swap1(g[2]);
            cell.a[3] = swap1(g[3]);
        }
        // edge lengths: edge i runs along coordinate axis ax[i], upwards or downwards
        int ax[3];
        double h[3], sg[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            ax[i] = (flags >> (13 + 3 * i)) & 3;
            sg[i] = (flags >> (15 + 3 * i)) & 1 ? -1.0 : 1.0;
            h[i] = m.bext[3 * (size_t)c + i];
        }
        {
            const double ih = recip(fmax(h[0], fmax(h[1], h[2])));
#pragma unroll
            for (int i = 0; i < 3; ++i) cell.gm[i] = (h[i] * ih) * (h[i] * ih);
        }
        // sorted vertex values (a network of 19 exchanges)
        double s[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) s[i] = cell.a[i];
        auto exch = [&](int i, int j) {
            const double x = min2(s[i], s[j]), y = max2(s[i], s[j]);
            s[i] = x;
            s[j] = y;
        };
        exch(0, 1); exch(2, 3); exch(4, 5); exch(6, 7);
        exch(0, 2); exch(1, 3); exch(4, 6); exch(5, 7);
        exch(1, 2); exch(5, 6);
        exch(0, 4); exch(1, 5); exch(2, 6); exch(3, 7);
        exch(2, 4); exch(3, 5);
        exch(1, 2); exch(3, 4); exch(5, 6);
        // a vertex value that is no number, or infinite, leaves no isoface (and the bulk flux), as in
        // k_surface; the clamps below would make a cut of it, and the sort has dropped it
        const double mag = fabs(cell.a[0]) + fabs(cell.a[1]) + fabs(cell.a[2]) + fabs(cell.a[4]);
        bool recon = s[7] - s[0] > A.flat_tol && mag + swap1(mag) < INFINITY;
        double iso = 0.0, un = 0.0;
        int rounds = 0;
        double S[3] = {0.0, 0.0, 0.0}, N[3] = {0.0, 0.0, 0.0};  // isoface centre (local) and normal per edge direction
        if (recon) {
#pragma unroll
            for (int e = 0; e < 9; ++e) {
                const double d = cell.a[kBoxEdge[e][1]] - cell.a[kBoxEdge[e][0]];
                cell.inv[e] = fabs(d) > kTiny ? recip(d) : -1.0 / kTiny;
                cell.up[e] = d > kTiny ? 1.0 : 0.0;
            }
            // bracket between consecutive sorted vertex values by bisection: at most three probes.  (A
            // guess that orders the probes, as in k_surface, saves none here: with 32 cells in a
            // wave, one of them nearly always needs the third.)
            const double target = 12.0 * aP;
            int il = 0, ih = 7;
            double lo = s[0], hi = s[7], ga = 12.0 - target, gb = -target;
            bool exact = false;
            while (ih - il > 1) {
                const int im = (il + ih) >> 1;  // 3, then 1 or 5, then 2, 4 or 6
                const double sodd = (im & 4) ? s[5] : ((im & 2) ? s[3] : s[1]);
                const double seven = (im & 4) ? ((im & 2) ? s[6] : s[4]) : s[2];
                const double sm = (im & 1) ? sodd : seven, gm = share12(cell, sm) - target;
                ++rounds;
                if (gm > 0.0) { il = im; lo = sm; ga = gm; }
                else if (gm < 0.0) { ih = im; hi = sm; gb = gm; }
                else { iso = sm; exact = true; break; }
            }
            // the faces for a wet pattern (of the open interval, or above a vertex value that is the
            // isovalue): isoface edges linear, areas quadratic in u = isovalue - xr
            double xr = 0.5 * (lo + hi);
            Edge2 E[3], R[3];  // each face's (first) isoface edge at xr, and its rate of change
            double ar[3][3];   // twice the wet area: ar[f][0] + u (ar[f][1] + u ar[f][2])
            bool wet0 = false, saddle[3], any_saddle = false;
            auto pattern = [&](double x) {
                bool w[8];
                double t[9], y[9], s[9], k[9], iv[9];
#pragma unroll
                for (int i = 0; i < 7; ++i) w[i] = cell.a[i] > x;
                cut_points(cell, x, t);
#pragma unroll
                for (int e = 0; e < 9; ++e) {
                    const bool cut = cut_edge(w, e);
                    y[e] = cell.up[e] - t[e];
                    s[e] = cut ? t[e] : 0.0;
                    k[e] = cut ? 1.0 : 0.0;
                    iv[e] = cut ? cell.inv[e] : 0.0;
                }
#pragma unroll
                for (int f = 0; f < 3; ++f) {
                    const int *n = kBoxFaceEdge[f];
                    const Edge2 e = face_edge(f, y, s, k);
                    // (a cut edge's wet part shrinks as the isovalue grows, whichever end is wet)
                    const Edge2 d{iv[n[0]] + iv[n[2]], iv[n[1]] + iv[n[3]], fabs(iv[n[0]]) - fabs(iv[n[2]]),
                                  fabs(iv[n[1]]) - fabs(iv[n[3]])};
                    ar[f][0] = fma(0.5, cross2(e, e), fabs(y[n[1]]) + fabs(y[n[2]]));
                    ar[f][1] = fma(0.5, cross2(e, d) + cross2(d, e), -(fabs(iv[n[1]]) + fabs(iv[n[2]])));
                    ar[f][2] = 0.5 * cross2(d, d);
                    E[f] = e;
                    R[f] = d;
                    saddle[f] = saddle_face(w, f);
                }
                wet0 = w[0];
                any_saddle = saddle[0] || saddle[1] || saddle[2];
                if (any_saddle) {
#pragma unroll
                    for (int f = 0; f < 3; ++f)
                        if (saddle[f]) {
                            Edge2 e2, d2;
                            second_edge(cell, f, wet0, x, e2, d2);
                            const Edge2 e = E[f] - e2, d = R[f] - d2;
                            ar[f][0] = fma(0.5, cross2(e, e) + cross2(e2, e2) - cross2(E[f], E[f]), ar[f][0]);
                            ar[f][1] = fma(0.5, (cross2(e, d) + cross2(d, e)) + (cross2(e2, d2) + cross2(d2, e2)) -
                                                    (cross2(E[f], R[f]) + cross2(R[f], E[f])), ar[f][1]);
                            ar[f][2] = fma(0.5, cross2(d, d) + cross2(d2, d2) - cross2(R[f], R[f]), ar[f][2]);
                            E[f] = e;
                            R[f] = d;
                        }
                }
            };
            auto edge_at = [&](int f, double v) {
                const Edge2 &e = E[f], &d = R[f];
                return Edge2{fma3(v, d.mp, e.mp), fma3(v, d.mq, e.mq), fma3(v, d.dp, e.dp), fma3(v, d.dq, e.dq)};
            };
            double u = 0.0;
            bool at_vertex = exact;
            if (!exact) {
                pattern(xr);
                ++rounds;
                // twelve times the wet share less its target, and its derivative
                auto G = [&](double v, double &dG) {
                    // sums over three edges and their rates, as perimeter()
                    auto sums = [&](const Edge2 *e, const Edge2 *d, Perimeter &s, Perimeter &ds) {
                        double l[3], dl[3];
#pragma unroll
                        for (int f = 0; f < 3; ++f) {
                            const double gp = cell.gm[(f + 1) % 3] * e[f].dp, gq = cell.gm[(f + 2) % 3] * e[f].dq;
                            const Root k = root(fma(gp, e[f].dp, gq * e[f].dq));
                            l[f] = k.s;
                            dl[f] = fma(gp, d[f].dp, gq * d[f].dq) * k.r;
                        }
                        s = Perimeter{l[0] + l[1] + l[2],
                                      {fma(l[2], e[2].mp, l[1] * e[1].mq), fma(l[0], e[0].mp, l[2] * e[2].mq),
                                       fma(l[1], e[1].mp, l[0] * e[0].mq)}};
                        ds = Perimeter{dl[0] + dl[1] + dl[2],
                                       {fma(l[2], d[2].mp, fma(dl[2], e[2].mp, fma(l[1], d[1].mq, dl[1] * e[1].mq))),
                                        fma(l[0], d[0].mp, fma(dl[0], e[0].mp, fma(l[2], d[2].mq, dl[2] * e[2].mq))),
                                        fma(l[1], d[1].mp, fma(dl[1], e[1].mp, fma(l[0], d[0].mq, dl[0] * e[0].mq)))}};
                    };
                    Perimeter s, ds;
                    const Edge2 ev[3] = {edge_at(0, v), edge_at(1, v), edge_at(2, v)};
                    sums(ev, R, s, ds);
                    if (any_saddle) {
#pragma unroll
                        for (int f = 0; f < 3; ++f)
                            if (saddle[f]) {
                                const int p = (f + 1) % 3, q = (f + 2) % 3;
                                Edge2 e, d;
                                second_edge(cell, f, wet0, xr + v, e, d);
                                const double gp = cell.gm[p] * e.dp, gq = cell.gm[q] * e.dq;
                                const Root k = root(fma(gp, e.dp, gq * e.dq));
                                const double dl = fma(gp, d.dp, gq * d.dq) * k.r;
                                s.l += k.s;
                                ds.l += dl;
                                s.m[p] = fma(k.s, e.mp, s.m[p]);
                                s.m[q] = fma(k.s, e.mq, s.m[q]);
                                ds.m[p] = fma(k.s, d.mp, fma(dl, e.mp, ds.m[p]));
                                ds.m[q] = fma(k.s, d.mq, fma(dl, e.mq, ds.m[q]));
                            }
                    }
                    const double L = s.l, dL = ds.l, *M = s.m, *dM = ds.m;
                    const double lt = L + swap1(L), dlt = dL + swap1(dL), il = recip(lt);
                    double g = 0.0, dg = 0.0;
#pragma unroll
                    for (int f = 0; f < 3; ++f) {
                        const double o = il * (M[f] + swap1(fma(2.0, L, -M[f])));
                        const double od = il * fma(-dlt, o, dM[f] + swap1(fma(2.0, dL, -dM[f])));
                        const double k = fma3(v, ar[f][2], ar[f][1]);
                        const double av = fma3(v, k, ar[f][0]);
                        const double dv = fma(v, ar[f][2], k);
                        g = fma(o, av, g);
                        dg = fma(od, av, fma(o, dv, dg));
                    }
                    dG = dg + swap1(dg);
                    return g + swap1(g) - target;
                };
                // Newton safeguarded by the bracket, as in k_surface; a Newton step that leaves the
                // bracket is replaced by the root of a cubic power law anchored at the end with the
                // smaller residual (to a float's accuracy: a guess as good), or bisection.  The value at
                // the bracket's upper end, the limit from below there, shows whether the sub-volume
                // jumps across alpha_P at that vertex value (vertices tied along an edge, or a corner
                // that joins across a saddle face).
                const double ulo = lo - xr, uhi = hi - xr;
                double ua = ulo, ub = uhi, up = uhi, dGp;
                bool conv = false;
                gb = G(uhi, dGp);
                const bool jump = gb > 0.0;
                u = fma(uhi - ulo, ga * recip(ga - gb), ulo);  // secant start
                const double shrt = 1e-3 * (uhi - ulo);
                while (!jump && rounds < A.max_rounds) {
                    double dG;
                    const double g = G(u, dG);
                    ++rounds;
                    if (fabs(g) <= 12.0 * A.root_tol) { conv = true; break; }  // g == 0 at 0
                    if (g > 0.0) { ua = u; ga = g; } else { ub = u; gb = g; }
                    double nu = fma(-g, recip(dG), u);
                    const bool newton = nu > ua && nu < ub;
                    if (!newton) {
                        const bool left = ga <= -gb;
                        const double q = (left ? ga : -gb) * recip(ga - gb);
                        const double w = (ub - ua) * (double)__builtin_amdgcn_exp2f(__builtin_amdgcn_logf((float)q) * (1.0f / 3.0f));
                        nu = left ? ua + w : ub - w;
                        if (!(nu > ua && nu < ub)) nu = 0.5 * (ua + ub);
                    }
                    // converged when the step is at round-off of the isovalue, or when a short Newton
                    // step leaves an error |G''| d^2 / (2 |G'|), G'' from the last two slopes, below an
                    // eighth of that; or when the bracket is
                    const double tolu = 2.0 * __DBL_EPSILON__ * max2(fabs(xr + nu), 1e-300);
                    const double d = nu - u;
                    const bool done = fabs(d) <= tolu ||
                                      (newton && fabs(d) <= shrt &&
                                       fabs(dG - dGp) * (d * d) <= 0.25 * tolu * fabs(dG * (u - up))) ||
                                      !(ub - ua > 2.0 * __DBL_EPSILON__ * max2(fabs(xr + ua), fabs(xr + ub)));
                    up = u;
                    dGp = dG;
                    u = nu;
                    if (done) { conv = true; break; }
                }
                if (jump) {
                    iso = hi;
                    at_vertex = true;
                } else {
                    if (!conv && r == 0) ++nonconv;
                    iso = xr + u;
                }
            }
            if (at_vertex) {  // the isoface is that of the pattern above the vertex value
                xr = iso;
                u = 0.0;
                pattern(xr);
            }
            // the isoface at the isovalue: apex (perimeter centroid), area vector (x2), and the centre
            // as the area-weighted fan centroid, taken relative to the apex
            // (the saddles' second edges enter each sum by a loop of their own)
            auto seconds = [&](auto &&use) {
#pragma unroll
                for (int f = 0; f < 3; ++f)
                    if (saddle[f]) {
                        Edge2 e2, d2;
                        second_edge(cell, f, wet0, xr + u, e2, d2);
                        use(f, e2);
                    }
            };
#pragma unroll
            for (int f = 0; f < 3; ++f) E[f] = edge_at(f, u);
            Perimeter ps = perimeter(cell, E);
            if (any_saddle) seconds([&](int f, const Edge2 &e) { add_edge(cell, f, e, ps); });
            double o2[3];
            apex(ps, o2);
            // twice (edge midpoint - apex) x (edge vector), components along f, p, q, from the entry cut
            // to the exit: on lane 1's faces against the walk's direction, on lane 0's (seen from
            // inside the cell) along it
            const double sn = r == 0 ? 1.0 : -1.0;
            auto cross3 = [&](int f, const Edge2 &e, double *k) {
                const int p = (f + 1) % 3, q = (f + 2) % 3;
                const double ap = e.mp - o2[p], aq = e.mq - o2[q];
                k[f] = fma(ap, e.dq, -(aq * e.dp));
                k[p] = o2[f] * e.dq;
                k[q] = -(o2[f] * e.dp);
            };
            double B[3];
            auto areas = [&](const Edge2 *e, double *B) {
                double k0[3], k1[3], k2[3];
                cross3(0, e[0], k0);
                cross3(1, e[1], k1);
                cross3(2, e[2], k2);
#pragma unroll
                for (int i = 0; i < 3; ++i) B[i] = k0[i] + k1[i] + k2[i];
            };
            areas(E, B);
            if (any_saddle)
                seconds([&](int f, const Edge2 &e) {
                    double k[3];
                    cross3(f, e, k);
#pragma unroll
                    for (int i = 0; i < 3; ++i) B[i] += k[i];
                });
#pragma unroll
            for (int i = 0; i < 3; ++i) B[i] *= sn;
            double ihn[3];  // normal over edge length: the area vector's weight per edge direction
            {
                double n2 = 0.0;
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    ihn[i] = recip(h[i]);
                    N[i] = (B[i] + swap1(B[i])) * ihn[i];
                    // both lanes add the same products in the same order
                    n2 = fma(N[i], N[i], n2);
                }
                const double len = sqrt(n2);
                recon = len > 0.0;
                const double rl = recon ? 1.0 / len : 0.0;
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    N[i] *= rl;
                    ihn[i] *= N[i];
                }
            }
            double acc[3] = {0.0, 0.0, 0.0}, ws = 0.0;
            auto centre = [&](int f, const Edge2 &e) {
                const int p = (f + 1) % 3, q = (f + 2) % 3;
                double k[3];
                cross3(f, e, k);
                const double wt = fma(k[2], ihn[2], fma(k[1], ihn[1], k[0] * ihn[0]));
                ws += wt;
                acc[f] = fma(wt, -o2[f], acc[f]);
                acc[p] = fma(wt, e.mp - o2[p], acc[p]);
                acc[q] = fma(wt, e.mq - o2[q], acc[q]);
            };
#pragma unroll
            for (int f = 0; f < 3; ++f) centre(f, E[f]);
            if (any_saddle) seconds(centre);
            // the lanes' area vectors point opposite ways around their own faces
            ws *= sn;
#pragma unroll
            for (int i = 0; i < 3; ++i) acc[i] *= sn;
            ws += swap1(ws);
            const double iw = recon ? recip(3.0 * ws) : 0.0;
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const double x = fma(iw, acc[i] - swap1(acc[i]), 0.5 * o2[i]);
                const double x0 = swap1(x);  // lane 1 mirrors lane 0's, so that both hold the same point
                S[i] = r ? 1.0 - x0 : x;
            }
        }
        if (recon) {
            double U[3];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const size_t at = ax[i] * nc + c;
                U[i] = A.U1 ? 0.5 * (A.U[at] + A.U1[at]) : A.U[at];
            }
            if constexpr (kInterp) {
                // the tetrahedron (cell centre, face mean, two face points) that holds the centre: the
                // face across which it lies furthest out of the middle, then that face's nearest edge;
                // the barycentric coordinates follow from the offsets alone.  Each lane takes two of
                // the face's four vertices.
                double y[3];
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    const double d = S[i] - 0.5, d0 = swap1(d);
                    y[i] = r ? d0 : d;
                }
                const double a0 = fabs(y[0]), a1 = fabs(y[1]), a2 = fabs(y[2]);
                const int fa = a0 >= a1 ? (a0 >= a2 ? 0 : 2) : (a1 >= a2 ? 1 : 2);
                const int p = fa == 2 ? 0 : fa + 1, q = fa == 0 ? 2 : fa - 1;
                auto pick = [&](int i) { return i == 0 ? y[0] : (i == 1 ? y[1] : y[2]); };
                const bool pq = fabs(pick(p)) >= fabs(pick(q));
                const int fb = pq ? p : q, fc = pq ? q : p;
                const double ya = pick(fa), yb = pick(fb), yc = pick(fc);
                const double t = 2.0 * fabs(ya), e = 2.0 * fabs(yb);
                const double end = 0.5 * (e + (r ? 2.0 * yc : -2.0 * yc));
                double w[2], us[3];
                int32_t k[2];
#pragma unroll
                for (int v = 0; v < 2; ++v) {
                    const int b = ((ya >= 0.0 ? 1 : 0) << fa) | (v << fb) | (r << fc);
                    w[v] = 0.25 * (t - e) + (v == (yb >= 0.0 ? 1 : 0) ? end : 0.0);
                    k[v] = m.cpt[8 * (size_t)c + ((kBoxCanon >> (4 * b)) & 7u)];
                }
                if (m.sten_n == 4) gather_velocity<4>(A, ax, k, w, us);
                else gather_velocity<8>(A, ax, k, w, us);
#pragma unroll
                for (int i = 0; i < 3; ++i) U[i] = fma(1.0 - t, U[i], us[i] + swap1(us[i]));
            }
            un = 0.0;
#pragma unroll
            for (int i = 0; i < 3; ++i) un = fma(N[i], sg[i] * U[i], un);
        }
        if (r == 0) {
            if (!recon) ++flat;
            rounds_max = max(rounds_max, rounds);
            if (A.tr.kind) A.tr.kind[c] = recon ? 1 : 2;
            if (recon) {
                if (A.tr.iso) A.tr.iso[c] = iso;
                if (A.tr.iters) A.tr.iters[c] = rounds;
                if (A.tr.rec) {
                    double *rr = A.tr.rec + 7 * (size_t)c;
#pragma unroll
                    for (int i = 0; i < 3; ++i) {
                        rr[ax[i]] = m.cxyz[24 * (size_t)c + ax[i]] + sg[i] * (S[i] * h[i]);
                        rr[3 + ax[i]] = sg[i] * N[i];
                    }
                    rr[6] = un;
                }
            }
        }
        // the lane's outflow faces
        const double dtc = cell_dt(m, A.dt_dom, A.dt, c);
        // a plane at rest counts as one that moves by less than any distance of its cell, one of infinite
        // speed as one that moves by more, and so, forwards, one whose speed is no number (as in k_surface)
        double ud = un * dtc;
        if (fabs(ud) < 1e-200) ud = 1e-200;
        if (!(ud < 1e200)) ud = 1e200;
        if (ud < -1e200) ud = -1e200;
        const double iud = recip(ud);
        double nl[3], d0 = 0.0;  // change of the distance along each local coordinate; distance at the origin
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            nl[i] = (r ? -N[i] : N[i]) * h[i];
            d0 = fma(-nl[i], S[i], d0);
        }
#pragma unroll
        for (int f = 0; f < 3; ++f) {
            const int32_t v = m.lface[6 * (size_t)c + (r ? kBoxFace[1][f] : kBoxFace[0][f])];
            if (v == kEmpty) continue;
            const int32_t fid = v >= 0 ? v : ~v;
            const double ph = A.phi1 ? flux_at<true>(A.phi, A.phi1, fid) : flux_at<false>(A.phi, A.phi1, fid);
            if (!((v >= 0 ? ph : -ph) > 0.0)) continue;
            double dv = aP * ph * dtc;
            if (recon) {
                const double np = nl[(f + 1) % 3], nq = nl[(f + 2) % 3];
                const double e0 = d0 + (min2(np, 0.0) + min2(nq, 0.0));
                const double hp = fabs(np), hq = fabs(nq);
                dv = ph * (dtc * rect_sweep(e0, min2(hp, hq), max2(hp, hq), ud, iud));
            }
            A.dvs[fid] = dv;
        }
    }
    if (A.want_stats) {
        for (int off = 32; off > 0; off >>= 1) {
            rounds_max = max(rounds_max, __shfl_xor(rounds_max, off));
            flat += __shfl_xor(flat, off);
            nonconv += __shfl_xor(nonconv, off);
        }
        if (__lane_id() == 0) {
            if (rounds_max) atomicMax(&A.counters[kCntMaxIter], rounds_max);
            if (flat) atomicAdd(&A.counters[kCntFlat], flat);
            if (nonconv) atomicAdd(&A.counters[kCntNonconv], nonconv);
        }
    }
}

}  // namespace

hipError_t launch_surface_box(const SurfArgs &a, const LaunchCfg &cfg, int us_mode, hipStream_t s) {
    long gs = ((long)a.cap + kGroups - 1) / kGroups;
    // persistent: pairs of lanes loop over the list, whose length is only known on the device (four
    // groups of one wave for each of the 256 threads that surface_blocks counts)
    gs = std::max(1L, std::min(gs, 4L * (cfg.surface_blocks > 0 ? cfg.surface_blocks : 2048)));
    if (us_mode == 1) hipLaunchKernelGGL((k_surface_box<true>), dim3((int)gs), dim3(kBlock), 0, s, a);
    else hipLaunchKernelGGL((k_surface_box<false>), dim3((int)gs), dim3(kBlock), 0, s, a);
    return hipGetLastError();
}

}  // namespace isoadv
