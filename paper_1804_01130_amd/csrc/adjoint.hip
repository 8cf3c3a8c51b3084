// Adjoint (vector-Jacobian product) of one isoAdvector step on gfx950, FP64.
//
// Given the adjoint of alpha_new, the step's inputs and its intermediates (vertex values, cell
// kinds, isovalues, face volumes dV and the update before bounding, as the traced forward step
// writes them), these launches produce the adjoints of alpha and phi:
//   prep       per cell: the update's round-off chop, the cells the bounding sweeps start from
//              (and their first corrections); per face buffers cleared
//   group      the bounding sweeps replayed with a tape (same arithmetic as the forward), then the
//              bounding step (end of Section 3.2) transposed, sweep by sweep in reverse; on a mesh of
//              more than 2^17 cells the first sweep is a launch on the whole grid (sweep), and its
//              reverse two (unsweep)
//   faces      per cell, a gather over its flux faces: transposes of the flux-form update and of
//              the bulk fluxes alpha_upwind phi dt; phi's adjoint through dV = phi * (dV/phi); and
//              the list of interface cells
//   surface    eight lanes per interface cell: the isoface, the sub-volume and the swept face
//              integrals (Eqs. tv .. intaplus) run backwards to the vertex values, the isovalue moving
//              with the volume constraint (implicit function); general polyhedra by forward-mode dual
//              numbers, sixteen lanes per (polyhedron, point value)
//   points     per point class, and cells, per cell: the transpose of the vertex interpolation
//              gathers the vertex adjoints to the stencil cells in a fixed order
#include <hip/hip_runtime.h>

#include <algorithm>

#include "device_common.h"

namespace isoadv {
namespace {

// ------------------------------------------------------------------------------- dual numbers
struct Dl {
    double v, d;  // value and derivative along one direction
};
__device__ __forceinline__ Dl operator+(Dl a, Dl b) { return {a.v + b.v, a.d + b.d}; }
__device__ __forceinline__ Dl operator-(Dl a, Dl b) { return {a.v - b.v, a.d - b.d}; }
__device__ __forceinline__ Dl operator*(Dl a, Dl b) { return {a.v * b.v, a.d * b.v + a.v * b.d}; }
__device__ __forceinline__ Dl operator*(double s, Dl a) { return {s * a.v, s * a.d}; }
__device__ __forceinline__ Dl operator/(Dl a, Dl b) {
    const double q = a.v / b.v;
    return {q, (a.d - q * b.d) / b.v};
}
__device__ __forceinline__ Dl dinv(Dl a) {
    const double q = 1.0 / a.v;
    return {q, -a.d * q * q};
}
__device__ __forceinline__ Dl dsqrt(Dl a) {
    const double r = sqrt(a.v);
    return {r, r > 0.0 ? 0.5 * a.d / r : 0.0};
}
__device__ __forceinline__ Dl dc(double x) { return {x, 0.0}; }

struct DV3 {
    Dl x, y, z;
};
__device__ __forceinline__ DV3 operator+(DV3 a, DV3 b) { return {a.x + b.x, a.y + b.y, a.z + b.z}; }
__device__ __forceinline__ DV3 operator-(DV3 a, DV3 b) { return {a.x - b.x, a.y - b.y, a.z - b.z}; }
__device__ __forceinline__ DV3 operator*(Dl s, DV3 a) { return {s * a.x, s * a.y, s * a.z}; }
__device__ __forceinline__ DV3 operator*(double s, DV3 a) { return {s * a.x, s * a.y, s * a.z}; }
__device__ __forceinline__ DV3 dv(D3 a) { return {dc(a.x), dc(a.y), dc(a.z)}; }
__device__ __forceinline__ Dl ddot(DV3 a, DV3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
__device__ __forceinline__ DV3 dcross(DV3 a, DV3 b) {
    return {a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x};
}
__device__ __forceinline__ Dl dnorm(DV3 a) { return dsqrt(ddot(a, a)); }
// Swept integral of a triangle (the forward kernel's construction in dual numbers): the wet
// fraction at time s is the area distribution of the distances at un*s; breakpoints clamped to
// the window; each piece integrated exactly (Simpson) on the branch of its midpoint.
__device__ __forceinline__ Dl dtri_piece(int br, Dl z, Dl e1, Dl e2, Dl e3, Dl r31, Dl r21, Dl r32) {
    if (br == 0) return dc(0.0);
    if (br == 3) return dc(1.0);
    if (br == 1) {
        const Dl u = z - e1;
        return (u * r31) * (u * r21);
    }
    const Dl u = e3 - z;
    return dc(1.0) - (u * r31) * (u * r32);
}

__device__ __forceinline__ Dl dtri_sweep(Dl d0, Dl d1, Dl d2, Dl un, double dt) {
    // sorted by compare-and-swap: a permutation, so at a tie each distance keeps its own rate
    // (a min and a max that both return the same member would count one vertex twice)
    Dl e1 = d0, e2 = d1, e3 = d2;
    auto order = [](Dl &x, Dl &y) {
        if (y.v < x.v) {
            const Dl t = x;
            x = y;
            y = t;
        }
    };
    order(e1, e2);
    order(e2, e3);
    order(e1, e2);
    const Dl r31 = e3.v > e1.v ? dinv(e3 - e1) : dc(0.0);
    const Dl r21 = e2.v > e1.v ? dinv(e2 - e1) : dc(0.0);
    const Dl r32 = e3.v > e2.v ? dinv(e3 - e2) : dc(0.0);
    auto branch = [&](double z) { return z < e1.v ? 0 : (z < e2.v ? 1 : (z < e3.v ? 2 : 3)); };
    if (un.v == 0.0) {
        const int br = branch(0.0);
        const Dl m = un * dc(0.5 * dt), b = un * dc(dt);
        return (dt / 6.0) * (dtri_piece(br, dc(0.0), e1, e2, e3, r31, r21, r32) +
                             4.0 * dtri_piece(br, m, e1, e2, e3, r31, r21, r32) +
                             dtri_piece(br, b, e1, e2, e3, r31, r21, r32));
    }
    const Dl inv = dinv(un);
    Dl s1 = e1 * inv, s2 = e2 * inv, s3 = e3 * inv;
    if (un.v < 0.0) {
        const Dl t = s1;
        s1 = s3;
        s3 = t;
    }
    const Dl bk[3] = {s1, s2, s3};
    Dl acc = dc(0.0), a0 = dc(0.0);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        Dl a1 = dc(dt);
        if (k < 3) a1 = bk[k].v <= 0.0 ? dc(0.0) : (bk[k].v >= dt ? dc(dt) : bk[k]);
        if (a1.v > a0.v) {
            const Dl m = 0.5 * (a0 + a1);
            const int br = branch(un.v * m.v);
            const Dl fa = dtri_piece(br, un * a0, e1, e2, e3, r31, r21, r32);
            const Dl fm = dtri_piece(br, un * m, e1, e2, e3, r31, r21, r32);
            const Dl fb = dtri_piece(br, un * a1, e1, e2, e3, r31, r21, r32);
            acc = acc + (1.0 / 6.0) * ((a1 - a0) * (fa + 4.0 * fm + fb));
            a0 = a1;
        }
    }
    return acc;
}

// ------------------------------------------------------------------------------------ kernels
// A chop or clamp that moves a value by at most this much only removes round-off (which side of a
// bound such a value lands on is decided by rounding order): its derivative passes through.  A
// larger one makes the value a constant.
constexpr double kRound = 1e-14;
constexpr uint64_t kCorrBit = 1ull << 3, kTouchedBit = 1ull << 19;  // bounding tape flags, slot k: << k

// General polyhedra: sixteen lanes per (polyhedron, direction); directions 0 .. 31 are point
// values, kBigIsoDir the isovalue; per polyhedron the rates G at [0, kBigIsoDir], C at kBigC + the
// same, then the jump and 6V (see k_adj_surface_big).
constexpr int kBGrp = 16, kBGrpPerBlock = 16, kBPts = 32;
constexpr int kBigIsoDir = 32, kBigC = 33, kBigJump = 66, kBigV6 = 67;
static_assert(kAdjGBig == 68, "per-polyhedron rates: 33 + 33 + 2");

// The update's round-off chop (a move of at most the bounding tolerance) passes the derivative
// unless it moves the value by more than kRound: then the update is a constant there.
__device__ __forceinline__ bool raw_chopped(double x, int clip, double tol) {
    return clip && ((x < -kRound && x >= -tol) || (x > 1.0 + kRound && x <= 1.0 + tol));
}

struct AdjArgs {
    DevMesh m;
    const double *alpha, *phi, *U;
    double dt;
    const double *dt_dom;
    double eps, tol;
    int clip, n_iter;
    // forward intermediates of this step
    const double *vert_alpha;  // [8 nc] (interface cells)
    const int32_t *kind;       // [nc]
    const double *iso;         // [nc] (reconstructed cells)
    const double *dV0;         // [nf] dV before bounding, per flux face
    const double *raw;         // [nc] update before chopping
    // adjoint in / out
    const double *abar_new;  // [nc]
    double *abar;            // [nc]
    double *phibar;          // [nf]
    AdjWork w;
};

// Bounding replayed with a tape, then reversed: one pass per forward sweep (phase B of sweep s fused
// with phase A of sweep s+1, as in the step's own sweeps; phase A of sweep 0 runs in k_adj_prep) and two
// per reversed sweep, each a turn of k_adj_group or a launch on the grid.  Tape per sweep s and listed
// cell (row s*nc + i, i its place in the sweep's list): a, need, sumcap, r, then cap and dV-now per slot;
// flags (64 bits, for up to 16 slots): bit 0 over, bit 1 r capped at 1, bit 2 sumcap > 0, bit 3+k slot k
// corrected, bit 19+k slot k read the running dV (corrected in an earlier sweep).  List order never
// affects a result: each listed cell writes only its own outflow faces and its own tape row, each touched
// cell only itself.
//
// Buffers that start every call at zero and are left so: the face marks (`touched`), two banks of
// cell marks (sweep s uses bank s&1: phase B of sweep s clears what phase A of sweep s+1 sets in the
// other bank), and three rotating correction buffers (sweep s writes s%3, sweep s+1 reads it and clears
// s-1's).

// Phase A of sweep s for listed cell P, row `row` of the sweep's list, with bounding state a: the
// correction of each outflow face and the tape row; the cells it touches come back through tsel.
template <int W>
__device__ __forceinline__ void adj_correct(const AdjArgs &A, int s, int32_t P, int row, double a, int32_t *mark,
                                            int32_t tsel[W + 1]) {
    constexpr int R = 4 + 2 * W;
    const int n = A.m.n_cells, nf = A.m.n_faces;
    const DevMesh &m = A.m;
    const AdjWork &w = A.w;
    const bool over = a > 1.0 + A.tol;
    const double dtc = cell_dt(m, A.dt_dom, A.dt, P);
    // all loads of one kind together, none behind a branch (an empty slot reads the last face)
    const double vP = m.vol[P];
    int32_t v[W], fid[W], nb[W], tch[W];
    double ph[W], cap[W], dvnow[W], dv0[W];
#pragma unroll
    for (int k = 0; k < W; ++k) {
        const int2 q = m.slot_pair[(size_t)P * W + k];
        v[k] = q.x;
        nb[k] = q.y;
        fid[k] = min(face_of(v[k]), nf - 1);
    }
#pragma unroll
    for (int k = 0; k < W; ++k) {
        ph[k] = A.phi[fid[k]];
        tch[k] = w.touched[fid[k]];
        dvnow[k] = w.dvcur[fid[k]];
        dv0[k] = A.dV0[fid[k]];
    }
    uint64_t flags = over ? 1 : 0;
    double sumcap = 0.0;
#pragma unroll
    for (int k = 0; k < W; ++k) {
        cap[k] = 0.0;
        const double outphi = seen_from(v[k], ph[k]);
        if (v[k] == kEmpty || !(outphi > 0.0)) {
            dvnow[k] = 0.0;
            continue;
        }
        if (tch[k]) flags |= kTouchedBit << k;
        else dvnow[k] = dv0[k];
        const double outv = seen_from(v[k], dvnow[k]);
        cap[k] = over ? outphi * dtc - outv : outv;
        if (cap[k] > 0.0) sumcap += cap[k];
    }
    const double need = over ? (a - 1.0) * vP : -a * vP;
    double r = 0.0;
    if (sumcap > 0.0) {
        flags |= 4;
        const double q = need / sumcap;
        if (q > 1.0) flags |= 2;
        r = fmin(q, 1.0);
    }
    if (atomicExch(&mark[P], 1) == 0) tsel[W] = P;
    double *delta = w.delta + (size_t)(s % 3) * nf;
#pragma unroll
    for (int k = 0; k < W; ++k) {
        if (!(sumcap > 0.0) || !(cap[k] > 0.0)) continue;
        flags |= kCorrBit << k;
        const double d = cap[k] * r;
        const double dd = seen_from(v[k], over ? d : -d);
        delta[fid[k]] = dd;
        w.dvcur[fid[k]] = dvnow[k] + dd;
        w.touched[fid[k]] = 1;
        if (nb[k] >= 0 && atomicExch(&mark[nb[k]], 1) == 0) tsel[k] = nb[k];
    }
    double *rec = w.tape + ((size_t)s * n + row) * R;
    rec[0] = a;
    rec[1] = need;
    rec[2] = sumcap;
    rec[3] = r;
#pragma unroll
    for (int k = 0; k < W; ++k) {
        rec[4 + k] = cap[k];
        rec[4 + W + k] = dvnow[k];
    }
    w.tflag[(size_t)s * n + row] = flags;
}

// Append `count` entries per thread to a device-wide list with one atomic per work-group (whole
// waves, at most 1024 threads, every one of which calls it).  Returns the index of this thread's first entry.
__device__ __forceinline__ int block_append(int count, int32_t *counter) {
    __shared__ int wsum[16];
    __shared__ int base;
    const int lane = __lane_id(), wid = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
    int incl = count;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(incl, o, 64);
        if (lane >= o) incl += y;
    }
    if (lane == 63) wsum[wid] = incl;
    __syncthreads();
    int before = 0, total = 0;
    for (int j = 0; j < nw; ++j) {
        const int t = wsum[j];
        before += j < wid ? t : 0;
        total += t;
    }
    if (threadIdx.x == 0) base = total > 0 ? atomicAdd(counter, total) : 0;
    __syncthreads();
    const int r = base + before + incl - count;
    __syncthreads();  // wsum and base are reused by the next call
    return r;
}

// Append the cells a lane's corrections touched to sweep s's touched list (every lane of the wave).
template <int W>
__device__ __forceinline__ void adj_append_touched(const AdjArgs &A, int s, const int32_t tsel[W + 1]) {
    int nt = 0;
#pragma unroll
    for (int k = 0; k <= W; ++k) nt += tsel[k] >= 0 ? 1 : 0;
    int b = wave_append(nt, &A.w.counters[kAdjT + s]);
    int32_t *T = A.w.tlist + (size_t)s * A.m.n_cells;
#pragma unroll
    for (int k = 0; k <= W; ++k)
        if (tsel[k] >= 0) T[b++] = tsel[k];
}

// per cell: start state of bounding (and phase A of its first sweep), lists, per-face adjoint
// buffers and phi_bar cleared
template <int W>
__global__ void __launch_bounds__(256) k_adj_prep(AdjArgs A) {
    const int n = A.m.n_cells;
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    // (a linear pass over the faces: through each cell's own slots it took 28.2 us, not 20.8, on 128x64x64)
    for (int64_t f = c; f < A.m.n_faces; f += (int64_t)gridDim.x * blockDim.x)
        A.phibar[f] = A.w.dVb[f] = A.w.phib[f] = A.w.dvcurbar[f] = 0.0;
    bool offend = false;
    double x = 0.0;
    if (c < n) {
        x = A.raw[c];
        if (A.clip) {
            if (x < 0.0 && x >= -A.tol) x = 0.0;
            else if (x > 1.0 && x <= 1.0 + A.tol) x = 1.0;
        }
        A.w.x[c] = x;
        offend = x > 1.0 + A.tol || x < -A.tol;
        // with no sweep, the final clip makes a cell out of bounds (beyond round-off) a constant
        const bool clamped = A.n_iter == 0 && A.clip && offend && (x < -kRound || x > 1.0 + kRound);
        const double xb = clamped ? 0.0 : A.abar_new[c];
        A.w.xbar[c] = xb;
        A.w.pv[c] = raw_chopped(A.raw[c], A.clip, A.tol) ? 0.0 : xb / A.m.vol[c];
        A.w.cflag[c] = clamped ? 1 : 0;
    }
    if (A.n_iter < 1) return;  // uniform
    const int row = block_append(offend ? 1 : 0, &A.w.counters[kAdjL]);
    int32_t tsel[W + 1];
#pragma unroll
    for (int k = 0; k <= W; ++k) tsel[k] = -1;
    if (offend) {
        A.w.list[row] = c;
        adj_correct<W>(A, 0, c, row, x, A.w.cmark, tsel);
    }
    adj_append_touched<W>(A, 0, tsel);
}

// A list's length (atomics filled it, perhaps in this kernel: not through the L1).
__device__ __forceinline__ int adj_count(const AdjArgs &A, int i) {
    return __hip_atomic_load(&A.w.counters[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Phase B of sweep s: every touched cell applies its faces' corrections in ascending face order
// (round-off chop; clamp on the last sweep); a cell still out of bounds runs phase A of sweep s+1.
// Over the cells b0 + threadIdx.x, and so on every `stride`.
template <int W>
__device__ __forceinline__ void adj_sweep(const AdjArgs &A, int s, int b0, int stride) {
    const int n = A.m.n_cells, nf = A.m.n_faces;
    const DevMesh &m = A.m;
    const AdjWork &w = A.w;
    const bool last = s == A.n_iter - 1;
    if (s >= 1) {  // sweep s-1's corrections were read before this sweep: clear them
        const int np = adj_count(A, kAdjL + s - 1);
        double *stale = w.delta + (size_t)((s - 1) % 3) * nf;
        for (int i = b0 + threadIdx.x; i < np; i += stride) {
            const int32_t P = w.list[(size_t)(s - 1) * n + i];
            const uint64_t flags = w.tflag[(size_t)(s - 1) * n + i];
#pragma unroll
            for (int k = 0; k < W; ++k)
                if (flags & (kCorrBit << k)) {
                    const int32_t v = m.slot_pair[(size_t)P * W + k].x;
                    stale[v >= 0 ? v : ~v] = 0.0;
                }
        }
    }
    const double *delta = w.delta + (size_t)(s % 3) * nf;
    const int32_t *T = w.tlist + (size_t)s * n;
    int32_t *mark = w.cmark + (size_t)(s & 1) * n;
    int32_t *mark_next = w.cmark + (size_t)((s + 1) & 1) * n;
    const int nT = adj_count(A, kAdjT + s);
    for (int i0 = b0; i0 < nT; i0 += stride) {  // whole waves iterate together
        const int i = i0 + threadIdx.x;
        bool again = false;
        int32_t Q = 0;
        double x = 0.0;
        if (i < nT) {
            Q = T[i];
            const double aq = w.x[Q], vq = m.vol[Q];
            int32_t v[W];
            double d[W];
#pragma unroll
            for (int k = 0; k < W; ++k) v[k] = m.slot_pair[(size_t)Q * W + k].x;
#pragma unroll
            for (int k = 0; k < W; ++k) d[k] = delta[min(face_of(v[k]), nf - 1)];
            double sum = 0.0;
#pragma unroll
            for (int k = 0; k < W; ++k)
                if (v[k] != kEmpty) sum += seen_from(v[k], d[k]);
            const double x0 = aq - sum / vq;
            x = x0;
            if (A.clip) {
                if (x < 0.0 && x >= -A.tol) x = 0.0;
                else if (x > 1.0 && x <= 1.0 + A.tol) x = 1.0;
                if (last) x = fmin(fmax(x, 0.0), 1.0);
            }
            if (fabs(x - x0) > kRound) w.cflag[Q] |= 1 << s;
            w.x[Q] = x;
            mark[Q] = 0;
            again = !last && (x > 1.0 + A.tol || x < -A.tol);
        }
        if (last) continue;  // uniform
        const int row = wave_append(again ? 1 : 0, &w.counters[kAdjL + s + 1]);
        int32_t tsel[W + 1];
#pragma unroll
        for (int k = 0; k <= W; ++k) tsel[k] = -1;
        if (again) {
            w.list[(size_t)(s + 1) * n + row] = Q;
            adj_correct<W>(A, s + 1, Q, row, x, mark_next, tsel);
        }
        adj_append_touched<W>(A, s + 1, tsel);
    }
}

// Reverse of sweep s, first half: the adjoint of each correction through the two cells it was
// applied to (a cell chopped or clamped in sweep s passes nothing back: it was a constant), and the
// chopped cells' adjoints zeroed.  The two sets are disjoint, so one kernel does both.  The forward
// replay is over: its face marks and this sweep's corrections are cleared here.
template <int W>
__device__ __forceinline__ void adj_unsweep_apply(const AdjArgs &A, int s, int t0, int stride) {
    const int n = A.m.n_cells, nf = A.m.n_faces;
    const DevMesh &m = A.m;
    const AdjWork &w = A.w;
    const int nl = adj_count(A, kAdjL + s), nt = adj_count(A, kAdjT + s);
    const int32_t *L = w.list + (size_t)s * n;
    const int32_t *T = w.tlist + (size_t)s * n;
    double *delta = w.delta + (size_t)(s % 3) * nf;
    for (int i = t0; i < nl; i += stride) {
        const int32_t P = L[i];
        const uint64_t flags = w.tflag[(size_t)s * n + i];
        const int32_t cP = w.cflag[P];
        const double xP = w.xbar[P], vP = m.vol[P];
        int2 q[W];
        int32_t co[W];
        double xo[W], vo[W];
#pragma unroll
        for (int k = 0; k < W; ++k) q[k] = m.slot_pair[(size_t)P * W + k];
#pragma unroll
        for (int k = 0; k < W; ++k) {
            const int32_t o = max(q[k].y, 0);
            co[k] = w.cflag[o];
            xo[k] = w.xbar[o];
            vo[k] = m.vol[o];
        }
#pragma unroll
        for (int k = 0; k < W; ++k) {
            if (!(flags & (kCorrBit << k))) continue;
            const int32_t f = face_of(q[k].x);
            double db = 0.0;
            if (!(cP & (1 << s))) db -= seen_from(q[k].x, xP) / vP;
            if (q[k].y >= 0 && !(co[k] & (1 << s))) db += seen_from(q[k].x, xo[k]) / vo[k];
            w.deltabar[f] = db;
            w.touched[f] = 0;
            delta[f] = 0.0;
        }
    }
    for (int j = t0; j < nt; j += stride) {
        const int32_t Q = T[j];
        if (w.cflag[Q] & (1 << s)) {
            w.xbar[Q] = 0.0;
            w.pv[Q] = 0.0;
        }
    }
}

// Reverse of sweep s, second half: through the corrections of each listed cell, to its bounding
// state, its outflow faces' fluxes and their dV (before bounding, or running from an earlier sweep).
template <int W>
__device__ __forceinline__ void adj_unsweep_correct(const AdjArgs &A, int s, int t0, int stride) {
    constexpr int R = 4 + 2 * W;
    const int n = A.m.n_cells;
    const DevMesh &m = A.m;
    const AdjWork &w = A.w;
    const int nl = adj_count(A, kAdjL + s);
    const int32_t *L = w.list + (size_t)s * n;
    for (int i = t0; i < nl; i += stride) {
        const int32_t P = L[i];
        const uint64_t flags = w.tflag[(size_t)s * n + i];
        const double *rec = w.tape + ((size_t)s * n + i) * R;
        const bool over = flags & 1;
        const double sumcap = rec[2], r = rec[3];
        const double dtc = cell_dt(m, A.dt_dom, A.dt, P);
        const double xP = w.xbar[P], vP = m.vol[P], raw = A.raw[P];
        int32_t v[W], fid[W];
        double cap[W], dlb[W], dvb[W], dV0b[W], phb[W];
#pragma unroll
        for (int k = 0; k < W; ++k) {
            cap[k] = rec[4 + k];
            v[k] = m.slot_pair[(size_t)P * W + k].x;
            fid[k] = min(face_of(v[k]), m.n_faces - 1);
        }
#pragma unroll
        for (int k = 0; k < W; ++k) {
            dlb[k] = w.deltabar[fid[k]];
            dvb[k] = w.dvcurbar[fid[k]];
            dV0b[k] = w.dVb[fid[k]];
            phb[k] = w.phib[fid[k]];
        }
        double capb[W], dvnb[W];
        double rb = 0.0;
#pragma unroll
        for (int k = 0; k < W; ++k) {
            capb[k] = 0.0;
            dvnb[k] = 0.0;
            if (!(flags & (kCorrBit << k))) continue;
            const double ddb = dlb[k] + dvb[k];
            const double d_b = seen_from(v[k], over ? ddb : -ddb);
            capb[k] = d_b * r;
            rb += d_b * cap[k];
            dvnb[k] = dvb[k];  // dvcur after = dV-now + correction
        }
        double needb = 0.0, sumcapb = 0.0;
        if ((flags & 4) && !(flags & 2)) {
            needb = rb / sumcap;
            sumcapb = -rb * r / sumcap;
        }
#pragma unroll
        for (int k = 0; k < W; ++k) {
            if (!(cap[k] > 0.0) || !(flags & 4)) continue;
            const int32_t f = fid[k];
            const double cb = capb[k] + sumcapb;
            const double outvb = over ? -cb : cb;
            if (over) w.phib[f] = phb[k] + seen_from(v[k], cb) * dtc;
            dvnb[k] += seen_from(v[k], outvb);
            if (flags & (kTouchedBit << k)) {
                w.dvcurbar[f] = dvnb[k];
            } else {
                w.dVb[f] = dV0b[k] + dvnb[k];
                w.dvcurbar[f] = 0.0;
            }
        }
        const double xb = xP + needb * (over ? vP : -vP);
        w.xbar[P] = xb;
        w.pv[P] = raw_chopped(raw, A.clip, A.tol) ? 0.0 : xb / vP;
    }
}

// The sweeps on the grid, and all from `first` on, forwards and back, in one launch, as in k_bound_group of the
// step (whose lists these are): a short list costs its launch and a chain of loads, so one work-group walks it
// alone; a long first list is shared, and so are the sweeps after it and those on the way back while their lists
// have more cells than a group has threads (Team).  An adjoint in us, one group whatever the length / this: calm
// 64x32x32 and 128x64x64 39.9 / 40.2 and 125.8 / 126.2, the violent start on 192x96x96 (1148 cells out of bounds)
// 406 / 364.  Step and adjoint, nine launches / one group / this, from fields out of bounds in every sweep:
// 64x32x32 (855) 266 / 289 / 207, (7.9 k) 296 / 1737 / 256, 128x64x64 (68 k) 780 / 10900 / 752, 256x128x128 (1.9 M)
// 4431 / 215000 / 5398, polyhedra 64x32x32 (3.8 k) 515 / 2060 / 464.
// A traced step and adjoint of 128x64x64 cells and the gradient of five 256x128 slab steps: nine launches
// 252 and 845 us, one group (and the gathers of k_adj_faces straight-line) 221 and 750, with the loads of
// a sweep's cell batched, none behind a branch, 205 and 660 (this kernel on the slab 18.3 -> 11.9; on the box
// 18.0, with 1024 threads and their 128 registers 27.5).
template <int W>
__global__ void __launch_bounds__(256) k_adj_sweep(AdjArgs A, int s) {
    adj_sweep<W>(A, s, blockIdx.x * blockDim.x, gridDim.x * blockDim.x);
}
template <int W>
__global__ void __launch_bounds__(256) k_adj_unsweep_apply(AdjArgs A, int s) {
    adj_unsweep_apply<W>(A, s, blockIdx.x * blockDim.x + threadIdx.x, gridDim.x * blockDim.x);
}
template <int W>
__global__ void __launch_bounds__(256) k_adj_unsweep_correct(AdjArgs A, int s) {
    adj_unsweep_correct<W>(A, s, blockIdx.x * blockDim.x + threadIdx.x, gridDim.x * blockDim.x);
}
constexpr int adj_group_threads(int W) { return W > 8 ? 256 : W > 4 ? 512 : 1024; }  // (its registers fit)
template <int W>
__global__ void __launch_bounds__(adj_group_threads(W)) k_adj_group(AdjArgs A, int first) {
    const int tid = threadIdx.x, bd = blockDim.x, n0 = adj_count(A, kAdjT + first);
    if (__builtin_expect(n0 <= kBoundAlone || gridDim.x <= 4, 1)) {
        if (blockIdx.x != 0) return;
        for (int s = first; s < A.n_iter; ++s) {
            adj_sweep<W>(A, s, 0, bd);
            __syncthreads();
        }
        for (int s = A.n_iter - 1; s >= first; --s) {
            adj_unsweep_apply<W>(A, s, tid, bd);
            __syncthreads();
            adj_unsweep_correct<W>(A, s, tid, bd);
            __syncthreads();
        }
        return;
    }
    // the phases: m sweeps, and two for each of them on the way back; the items of one, and its part i of `tiles`
    const int m = A.n_iter - first;
    const auto sweep = [&](int p) { return p < m ? first + p : A.n_iter - 1 - (p - m) / 2; };
    const auto items = [&](int p) { return adj_count(A, (p < m ? kAdjT : kAdjL) + sweep(p)); };
    const auto part = [&](int p, int i, int tiles, int width) {
        const int s = sweep(p), b0 = i * width, stride = tiles * width;
        if (tid >= width) return;
        if (p < m) adj_sweep<W>(A, s, b0, stride);
        else if (((p - m) & 1) == 0) adj_unsweep_apply<W>(A, s, b0 + tid, stride);
        else adj_unsweep_correct<W>(A, s, b0 + tid, stride);
    };
    Team *t = reinterpret_cast<Team *>(A.w.counters + kAdjTeam);
    const int tiles0 = team_tiles(n0);
    bool lead = false;
    int p = 0;
    for (uint32_t sum = tiles0;;) {
        const bool over = team_work(t, tiles0, lead, [&](int i) {
            const bool f = team_load(&t->word) == 0;  // the first phase
            const int n = f ? n0 : team_load(&t->arg[1]), tiles = team_tiles(n);
            part(f ? 0 : team_load(&t->arg[0]), i, tiles, team_width(n, tiles));
        });
        if (over) {
            team_leave(t);
            return;
        }
        if (!lead) {
            __builtin_amdgcn_s_sleep(4);
            continue;
        }
        team_close(t, sum);
        int n = 0;
        for (++p; p < 3 * m && (n = items(p)) <= bd; ++p) {
            part(p, 0, 1, bd);
            __syncthreads();
        }
        if (p == 3 * m) break;
        if (tid == 0) {
            t->arg[0] = p;
            t->arg[1] = n;
        }
        team_open(t, team_tiles(n));
        sum += team_tiles(n);
    }
    team_dismiss(t);
    team_leave(t);
}

// per cell: transposes of the update (through the round-off chop) and of the bulk fluxes
template <int W>
__device__ __forceinline__ void adj_faces_cell(const AdjArgs &A, int c) {
    const int n = A.m.n_cells;
    const DevMesh &m = A.m;
    // all loads of one kind together, none behind a branch (an empty slot reads the last face, a
    // boundary one cell 0): 43.1 -> 23.7 us on 128x64x64 cells
    int32_t v[W], o[W];
#pragma unroll
    for (int k = 0; k < W; ++k) {
        v[k] = m.slot_face[(size_t)k * n + c];
        o[k] = m.slot_nbr[(size_t)k * n + c];
    }
    double ph[W], db[W], pv[W], d0[W], pb[W];
#pragma unroll
    for (int k = 0; k < W; ++k) {
        const int32_t f = min(face_of(v[k]), m.n_faces - 1);
        ph[k] = A.phi[f];
        db[k] = A.w.dVb[f];
        pv[k] = A.w.pv[max(o[k], 0)];
        d0[k] = pb[k] = 0.0;
        if (v[k] >= 0) {
            d0[k] = A.dV0[f];
            pb[k] = A.w.phib[f];
        }
    }
    // adjoint of the update before its round-off chop, and the same over the volume (kept per cell
    // by the kernels that change it, so a neighbour costs one load)
    const double bc = raw_chopped(A.raw[c], A.clip, A.tol) ? 0.0 : A.w.xbar[c];
    const double Vc = m.vol[c];
    const bool recon = A.kind[c] == 1;
    const double dtc = cell_dt(m, A.dt_dom, A.dt, c);
    double acc = bc;
#pragma unroll
    for (int k = 0; k < W; ++k) {
        if (v[k] == kEmpty) continue;
        const int32_t f = face_of(v[k]);
        // alpha_raw(owner) -= dV/V_owner, alpha_raw(neighbour) += dV/V_neighbour
        const double po = o[k] >= 0 ? pv[k] : 0.0;
        const double dvb = (v[k] >= 0 ? -bc / Vc + po : -po + bc / Vc) + db[k];
        if (seen_from(v[k], ph[k]) > 0.0) {
            if (recon) A.w.vbar[f] = dvb * ph[k];  // dV = phi * (swept integral of the interface cell)
            else acc += dvb * ph[k] * dtc;         // dV = alpha_c phi dt
        }
        if (v[k] >= 0) A.phibar[f] = (ph[k] != 0.0 ? dvb * (d0[k] / ph[k]) : 0.0) + pb[k];
    }
    A.abar[c] = acc;
}

// per cell: transposes of the update and the bulk fluxes; the interface cells' work list
template <int W>
__global__ void __launch_bounds__(256) k_adj_faces(AdjArgs A) {
    const int n = A.m.n_cells;
    const int c = xcd_block(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;  // contiguous ranges per XCD
    if (c < n) adj_faces_cell<W>(A, c);
    int nbig = 0;  // a general polyhedron: every point value and the isovalue (kBigIsoDir)
    const bool cut = c < n && A.kind[c] == 1, big = cut && A.m.cbig && A.m.cbig[c] >= 0;
    if (big) {
        const int bi = A.m.cbig[c];
        nbig = A.m.bv_ptr[bi + 1] - A.m.bv_ptr[bi] + 1;
    }
    const int b = block_append(cut && !big ? 1 : 0, &A.w.counters[kAdjCells]);
    if (cut && !big) A.w.clist[b] = c;
    if (!A.m.cbig) return;  // uniform: no polyhedra in this mesh
    int bb = block_append(nbig, &A.w.counters[kAdjDirsBig]);
    for (int d = 0; d + 1 < nbig; ++d) A.w.dlist_big[bb++] = ((int64_t)c << 6) | d;
    if (nbig) A.w.dlist_big[bb] = ((int64_t)c << 6) | kBigIsoDir;
}

// ------------------------------------------------------------------------ interface cells (8 lanes)
// Rates of a triangle's swept integral with its vertices' distances and the normal speed: the integral
// over the window of the rates of G(un s), G the triangle's area distribution, piece by piece between
// its breakpoints (their integrands are quadratic, so the moments below are exact), and at a breakpoint
// where G jumps (three equal distances) the jump times the breakpoint's rate.
struct TriRates {
    double p0, p1, p2, pu;
};
__device__ __forceinline__ TriRates tri_rates(double d0, double d1, double d2, double un, double dt) {
    double e1 = d0, e2 = d1, e3 = d2;
    int i1 = 0, i2 = 1, i3 = 2;
    auto order = [](double &x, double &y, int &ix, int &iy) {
        const bool swap = y < x;
        const double t = swap ? y : x, u = swap ? x : y;
        const int it = swap ? iy : ix, iu = swap ? ix : iy;
        x = t;
        y = u;
        ix = it;
        iy = iu;
    };
    order(e1, e2, i1, i2);
    order(e2, e3, i2, i3);
    order(e1, e2, i1, i2);
    const double r31 = e3 > e1 ? 1.0 / (e3 - e1) : 0.0;
    const double r21 = e2 > e1 ? 1.0 / (e2 - e1) : 0.0;
    const double r32 = e3 > e2 ? 1.0 / (e3 - e2) : 0.0;
    double q1 = 0.0, q2 = 0.0, q3 = 0.0, qu = 0.0;
    const double inv = un != 0.0 ? 1.0 / un : 0.0;
    const bool up = un > 0.0;
    // breakpoints in the order they are met, clamped to the window (a speed of zero meets none)
    const double sa = up ? e1 * inv : e3 * inv, sb = e2 * inv, sc = up ? e3 * inv : e1 * inv;
    auto clamp = [&](double x) { return un == 0.0 || x <= 0.0 ? 0.0 : (x >= dt ? dt : x); };
    const double bk[4] = {clamp(sa), clamp(sb), clamp(sc), dt};
    double jump[3] = {0.0, 0.0, 0.0};
    double a0 = 0.0;
    int prev = -1;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const double a1 = bk[k];
        if (a1 > a0) {
            const double z = un * (0.5 * (a0 + a1));
            const bool rising = z < e2;  // on the branch of the smallest distance, else of the largest
            double fa = z < e1 ? 0.0 : 1.0, fb = fa;
            if (z >= e1 && z < e3) {
                const double z0 = un * a0, h = a1 - a0;
                const double u0 = rising ? z0 - e1 : e3 - z0, u1 = u0 + (rising ? un : -un) * h;
                const double rB = rising ? r21 : r32, kk = r31 * rB;
                const double m1 = h * (u0 + u1), m2 = (1.0 / 3.0) * h * (u0 * u0 + u0 * u1 + u1 * u1);
                const double ms = (1.0 / 3.0) * h * (u0 * (a0 + a0 + a1) + u1 * (a0 + a1 + a1));
                const double self = kk * (m2 * (r31 + rB) - m1), other = -kk * r31 * m2;
                q1 += rising ? self : other;
                q3 += rising ? other : self;
                q2 -= kk * rB * m2;
                qu += kk * ms;
                const double g0 = (u0 * r31) * (u0 * rB), g1 = (u1 * r31) * (u1 * rB);
                fa = rising ? g0 : 1.0 - g0;
                fb = rising ? g1 : 1.0 - g1;
            }
#pragma unroll
            for (int j = 0; j < 3; ++j)
                if (j < k && j == prev) jump[j] -= fa;
            if (k < 3) jump[k < 3 ? k : 0] += fb;
            prev = k;
            a0 = a1;
        }
    }
    // (a breakpoint clamped to the window's end does not move)
    const double ja = sa < dt ? jump[0] * inv : 0.0, jb = sb < dt ? jump[1] * inv : 0.0, jc = sc < dt ? jump[2] * inv : 0.0;
    q1 += up ? ja : jc;
    q2 += jb;
    q3 += up ? jc : ja;
    qu -= ja * sa + jb * sb + jc * sc;
    auto back = [](bool first, double a, bool second, double b, double c) { return first ? a : (second ? b : c); };
    return {back(i1 == 0, q1, i2 == 0, q2, q3), back(i1 == 1, q1, i2 == 1, q2, q3), back(i1 == 2, q1, i2 == 2, q2, q3), qu};
}

// One edge of the isoface: the face's wet loop enters at cut s0 (between wet vertex qn and a dry one)
// and left at cut s1 (from wet vertex qx).
struct IsoEdge {
    D3 s0, s1, t0, t1, qn, qx;      // cuts; wet to dry along their edges; wet ends
    double lam0, lam1, g0, g1;      // cut = wet end + lam t; rate of lam with the isovalue
    int n, dn, x, dx;               // the cell's vertices: wet and dry end of the entry, of the exit
    bool on;
};

// adjoints of the edge's cuts from those of o's sums, (s0 + s1) |s1 - s0| / 2 and |s1 - s0|, and of
// the area vector s0 x s1
__device__ __forceinline__ void iso_edge_back(const IsoEdge &S, D3 oab, double olb, D3 csb, D3 &s0b, D3 &s1b) {
    const D3 d = S.s1 - S.s0;
    const double l = norm3(d);
    const double lb = 0.5 * dot(oab, S.s0 + S.s1) + olb, q = l > 0.0 ? lb / l : 0.0;
    const D3 half = 0.5 * l * oab;
    s0b = s0b + half - q * d + cross(S.s1, csb);
    s1b = s1b + half + q * d + cross(csb, S.s0);
}

// Interface cells: adjoints of the vertex values and of alpha through the cell's isoface, by reverse
// accumulation; one group of eight lanes per cell, one lane per face, in the forward kernel's
// construction.  Two functions of the vertex values and the isovalue are differentiated: six times the
// sub-volume (G) and the faces' adjoint-weighted swept integrals (C), whose rate with the normal, the
// centre and the apex runs back over the same isoface edges.
// Bound by latency: one chain of some 2500 FP64 instructions per cell.  A forward-mode pass per
// direction (up to nine a cell, eight lanes each) took 72.9 us on 128x64x64 cells and 13.3 on a slab of
// 256x128; this takes 20.7 and 10.7.  It holds 376 registers, one wave per SIMD; with two (256
// registers, the rest spilled) 25.8 and 12.9.
__global__ void __launch_bounds__(64) k_adj_surface(AdjArgs A) {
    const DevMesh &m = A.m;
    const int lv = threadIdx.x & (kLanes - 1);
    const int ngrp = (gridDim.x * blockDim.x) / kLanes;
    const int ncell = A.w.counters[kAdjCells];
    const D3 Z{0, 0, 0};
    int fv[4];
    lane_face_loop(lv, fv);
    bool face_on = lv < 6;
    for (int g = (blockIdx.x * blockDim.x + threadIdx.x) / kLanes; g < ncell; g += ngrp) {
        const int c = A.w.clist[g];
        if (m.cloop) {  // cells other than hexahedra: the cell's own face loops, as in the step
            const int32_t L = lv < 6 ? m.cloop[6 * (size_t)c + lv] : 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) fv[i] = (L >> (3 * i)) & 7;
            face_on = (L >> 12) & 1;
        }
        const double aP = A.alpha[c];
        const double V6 = 6.0 * m.vol[c];
        const double dtc = cell_dt(m, A.dt_dom, A.dt, c);
        const double iso = A.iso[c];
        const D3 U{A.U[c], A.U[m.n_cells + c], A.U[2 * (size_t)m.n_cells + c]};
        const bool planar = (m.cflags[c] >> min(lv, 5)) & 1;
        const double *cx = m.cxyz + 24 * (size_t)c + 3 * lv;
        D3 xv{cx[0], cx[1], cx[2]};
        const double av = A.vert_alpha[8 * (size_t)c + lv];
        // the face's adjoint weight: zero unless the flux leaves the cell
        const int32_t sv = face_on ? m.lface[6 * (size_t)c + lv] : kEmpty;
        double wgt = 0.0;
        if (sv != kEmpty) {
            const int32_t fid = sv >= 0 ? sv : ~sv;
            const double ph = A.phi[fid];
            if ((sv >= 0 ? ph : -ph) > 0.0) wgt = A.w.vbar[fid];
        }
        xv = xv - 0.125 * grp_sum3(xv);
        D3 q[4];
        int wet = 0, ids = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            q[i] = D3{grp_get(xv.x, fv[i]), grp_get(xv.y, fv[i]), grp_get(xv.z, fv[i])};
            wet |= (grp_get(av, fv[i]) > iso ? 1 : 0) << i;
            ids |= fv[i] << (4 * i);
        }
        if (!face_on) wet = 0;
        // the face's isoface edges: one, or two on a saddle
        const int entries = ~wet & ((wet >> 1) | (wet << 3)) & 15;
        auto iso_edge = [&](int on) {
            IsoEdge S;
            S.on = on != 0;
            const int e = S.on ? __ffs(on) - 1 : 0;  // loop position of the dry end
            const int l = (wet >> ((e + 3) & 3)) & 1 ? e + 3 : ((wet >> ((e + 2) & 3)) & 1 ? e + 2 : e + 1);
            auto id = [&](int i) { return (ids >> (4 * (i & 3))) & 15; };
            S.dn = id(e);
            S.n = id(e + 1);
            S.x = id(l);
            S.dx = id(l + 1);
            auto at = [&](int v) { return D3{grp_get(xv.x, v), grp_get(xv.y, v), grp_get(xv.z, v)}; };
            S.qn = at(S.n);
            S.qx = at(S.x);
            S.t0 = at(S.dn) - S.qn;
            S.t1 = at(S.dx) - S.qx;
            const double an = grp_get(av, S.n), ax = grp_get(av, S.x);
            const double D0 = grp_get(av, S.dn) - an, D1 = grp_get(av, S.dx) - ax;
            S.g0 = S.on ? 1.0 / D0 : 0.0;
            S.g1 = S.on ? 1.0 / D1 : 0.0;
            S.lam0 = (iso - an) * S.g0;
            S.lam1 = (iso - ax) * S.g1;
            S.s0 = S.qn + S.lam0 * S.t0;
            S.s1 = S.qx + S.lam1 * S.t1;
            return S;
        };
        const IsoEdge E0 = iso_edge(entries);
        const bool saddles = __any((entries & (entries - 1)) != 0);
        IsoEdge E1{};
        if (saddles) E1 = iso_edge(entries & (entries - 1));
        auto edges = [&](auto body) {
            if (E0.on) body(E0, 0);
            if (saddles && E1.on) body(E1, 1);
        };
        // the isoface's sums and apex
        D3 cseg = Z, oacc = Z;
        double oL = 0.0;
        edges([&](const IsoEdge &S, int) {
            const double l = norm3(S.s1 - S.s0);
            cseg = cseg + cross(S.s0, S.s1);
            oacc = oacc + (0.5 * l) * (S.s0 + S.s1);
            oL += l;
        });
        const D3 lseg = cseg;  // the face's own
        cseg = grp_sum3(cseg);
        oacc = grp_sum3(oacc);
        oL = grp_sum(oL);
        D3 o = Z;
        if (oL > 0.0) {
            o = (1.0 / oL) * oacc;
        } else {  // no edge has a length: the mean of their ends
            D3 os = Z;
            double ns = 0.0;
            edges([&](const IsoEdge &S, int) {
                os = os + S.s0;
                ns += 1.0;
            });
            os = grp_sum3(os);
            ns = grp_sum(ns);
            if (ns > 0.0) o = (1.0 / ns) * os;
        }
        // the wet part of the face: its area vector C (x2) and, on a face that is not planar, the apex
        // over its loop; six times the sub-volume
        D3 C = Z - lseg, ap = q[0], pacc = Z;
        double pl = 0.0;
        if (wet) {
            auto side = [&](bool on, D3 u, D3 v) {
                if (on) C = C + cross(u, v);
                if (on && !planar) {
                    const double l = norm3(v - u);
                    pacc = pacc + (0.5 * l) * (u + v);
                    pl += l;
                }
            };
#pragma unroll
            for (int i = 0; i < 4; ++i) side((wet >> i) & (wet >> ((i + 1) & 3)) & 1, q[i], q[(i + 1) & 3]);
            edges([&](const IsoEdge &S, int) {
                side(true, S.qx, S.s1);
                side(true, S.s0, S.qn);
                if (!planar) {
                    const double l = norm3(S.s1 - S.s0);
                    pacc = pacc + (0.5 * l) * (S.s0 + S.s1);
                    pl += l;
                }
            });
            if (!planar && pl > 0.0) ap = (1.0 / pl) * pacc;
        }
        const double v6 = grp_sum(wet ? dot(ap, C) : 0.0) + dot(o, cseg);
        const double nrm = norm3(cseg);
        // cut adjoints along their edges: of G (yg) and of C (yc), entry and exit of each edge
        double yg[2][2] = {{0.0, 0.0}, {0.0, 0.0}}, yc[2][2] = {{0.0, 0.0}, {0.0, 0.0}};
        D3 oab = Z, csb = Z;
        double olb = 0.0;
        const double invL = oL > 0.0 ? 1.0 / oL : 0.0;
        if (nrm > 0.0) {
            const D3 n = (1.0 / nrm) * cseg;
            D3 acc = Z;
            double ws = 0.0;
            edges([&](const IsoEdge &S, int) {
                const double wt = dot(cross(S.s0 - o, S.s1 - o), n);
                acc = acc + wt * (o + S.s0 + S.s1);
                ws += wt;
            });
            acc = grp_sum3(acc);
            ws = grp_sum(ws);
            const double inv3w = 1.0 / (3.0 * ws);
            const D3 xS = inv3w * acc;
            const double un = dot(U, n);
            // the swept integrals' rates with the distances of the face's vertices and apex, and the speed
            D3 xb = Z, nb = Z;
            if (wgt != 0.0) {
                const D3 B = sel3(planar, q[0], 0.25 * (q[0] + q[1] + q[2] + q[3]));
                const double dB = dot(B - xS, n);
                double d[4], area[4], db[4] = {0.0, 0.0, 0.0, 0.0}, dBb = 0.0, unb = 0.0, Af = 0.0;
                D3 x[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) x[i] = sel3(planar, q[(i + 1) & 3], q[i]);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    d[i] = dot(x[i] - xS, n);
                    area[i] = i < 2 || !planar ? 0.5 * norm3(cross(x[i] - B, x[(i + 1) & 3] - B)) : 0.0;
                    Af += area[i];
                }
#pragma unroll 1
                for (int t = planar ? 2 : 4; t > 0; --t) {  // triangle (B, x0, x1), then the next
                    const TriRates r = tri_rates(dB, d[0], d[1], un, dtc);
                    dBb += area[0] * r.p0;
                    unb += area[0] * r.pu;
                    const double b0 = db[0] + area[0] * r.p1, b1 = db[1] + area[0] * r.p2;
                    const double ta = area[0], td = d[0];
#pragma unroll
                    for (int i = 0; i < 3; ++i) {
                        area[i] = area[i + 1];
                        d[i] = d[i + 1];
                    }
                    area[3] = ta;
                    d[3] = td;
                    db[0] = b1;
                    db[1] = db[2];
                    db[2] = db[3];
                    db[3] = b0;
                }
                // (after two turns position i holds vertex i + 2, after four it holds vertex i)
                const double wA = wgt / Af;
                D3 sx = dBb * (B - xS);
                double sd = dBb;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    sx = sx + db[i] * (sel3(planar, x[(i + 2) & 3], x[i]) - xS);
                    sd += db[i];
                }
                nb = wA * (sx + unb * U);
                xb = (-(wA * sd)) * n;
            }
            xb = grp_sum3(xb);
            const D3 accb = inv3w * xb;
            const double wsb = -3.0 * dot(accb, xS);
            D3 ob = Z;
            D3 c0[2] = {Z, Z}, c1[2] = {Z, Z};
            edges([&](const IsoEdge &S, int k) {
                const D3 P = S.s0 - o, Q = S.s1 - o, cr = cross(P, Q);
                const double wt = dot(cr, n), wtb = dot(accb, o + S.s0 + S.s1) + wsb;
                const D3 wa = wt * accb, pb = wtb * cross(Q, n), qb = wtb * cross(n, P);
                c0[k] = wa + pb;
                c1[k] = wa + qb;
                ob = ob + wa - pb - qb;
                nb = nb + wtb * cr;
            });
            ob = grp_sum3(ob);
            nb = grp_sum3(nb);
            oab = invL * ob;
            olb = -dot(oab, o);
            csb = (1.0 / nrm) * (nb - dot(n, nb) * n);
            edges([&](const IsoEdge &S, int k) {
                iso_edge_back(S, oab, olb, csb, c0[k], c1[k]);
                yc[k][0] = dot(c0[k], S.t0);
                yc[k][1] = dot(c1[k], S.t1);
            });
        }
        // G: o . cseg, and each face's apex . C
        const D3 goa = invL * cseg;
        const double gol = -dot(goa, o);
        const D3 pab = planar || !(pl > 0.0) ? Z : (1.0 / pl) * C;
        const double plb = -dot(pab, ap);
        edges([&](const IsoEdge &S, int k) {
            D3 s0b = cross(ap, S.s1 - S.qn), s1b = cross(ap, S.qx - S.s0);
            iso_edge_back(S, goa, gol, o, s0b, s1b);
            if (!planar) {
                auto side = [&](D3 u, D3 v, D3 &ub, D3 &vb) {
                    const D3 d = v - u;
                    const double l = norm3(d), lb = 0.5 * dot(pab, u + v) + plb, f = l > 0.0 ? lb / l : 0.0;
                    ub = ub + 0.5 * l * pab - f * d;
                    vb = vb + 0.5 * l * pab + f * d;
                };
                D3 fixed = Z;
                side(S.qx, S.s1, fixed, s1b);
                side(S.s1, S.s0, s1b, s0b);
                side(S.s0, S.qn, s0b, fixed);
            }
            yg[k][0] = dot(s0b, S.t0);
            yg[k][1] = dot(s1b, S.t1);
        });
        // to the isovalue and the vertex values: cut = wet end + lam t, lam = (iso - a_wet) / (a_dry - a_wet)
        double gi = 0.0, ci = 0.0;
        double gv[8], cv[8];
#pragma unroll
        for (int v = 0; v < 8; ++v) gv[v] = cv[v] = 0.0;
        edges([&](const IsoEdge &S, int k) {
            auto cut = [&](int w, int d, double lam, double rate, double y, double z) {
                const double a = rate * y, b = rate * z;
                gi += a;
                ci += b;
#pragma unroll
                for (int v = 0; v < 8; ++v) {
                    const double f = v == w ? lam - 1.0 : (v == d ? -lam : 0.0);
                    gv[v] += f * a;
                    cv[v] += f * b;
                }
            };
            cut(S.n, S.dn, S.lam0, S.g0, yg[k][0], yc[k][0]);
            cut(S.x, S.dx, S.lam1, S.g1, yg[k][1], yc[k][1]);
        });
        gi = grp_sum(gi);
        ci = grp_sum(ci);
        double G = 0.0, Cv = 0.0;  // vertex lv's
#pragma unroll
        for (int v = 0; v < 8; ++v) {
            const double a = grp_sum(gv[v]), b = grp_sum(cv[v]);
            G = v == lv ? a : G;
            Cv = v == lv ? b : Cv;
        }
        // The isovalue moves with the volume constraint, so the adjoint of vertex value v is its rate at
        // fixed isovalue plus the isovalue's rate along v, -G_v / G_iso, times the rate along the
        // isovalue; alpha_P's is V6 / G_iso times that.  At a jump of the sub-volume the isovalue is the
        // jumping vertex's value and moves with it (rate 1 for that one, 0 otherwise and for alpha_P).
        const bool jump = fabs(v6 - aP * V6) > 1e-9 * V6;
        const uint64_t hit = __ballot(jump && av == iso);
        const int mvert = (int)((hit >> (__lane_id() & ~(kLanes - 1))) & 0xFF);
        double xdot, adot;
        if (jump) {
            xdot = mvert && __ffs(mvert) - 1 == lv ? 1.0 : 0.0;
            adot = 0.0;
        } else {
            xdot = gi != 0.0 ? -G / gi : 0.0;
            adot = gi != 0.0 ? V6 / gi : 0.0;
        }
        double *gb = A.w.gbuf + (size_t)kAdjG * c;
        gb[lv] = Cv + xdot * ci;
        if (lv == 0) gb[8] = adot * ci;
    }
}

// ------------------------------------------------------------------ general polyhedra (16 lanes)
// One group of sixteen lanes per (polyhedron, direction), lane lf on the cell's face lf, as in the
// forward polyhedron kernel: the cell's points (relative to their mean) and vertex values sit in
// LDS, the vertex values recomputed through the same stencils in the same order, so they are the
// forward's bits.  Directions 0 .. nv-1 are the points' values, kBigIsoDir the isovalue; the rates
// are stored per polyhedron: G (six times the sub-volume) at [0, kBigIsoDir], C (the faces'
// adjoint-weighted swept integrals) at kBigC + [0, kBigIsoDir], then the jump and 6V.

struct BPt {
    double x, y, z, a;
};
__device__ __forceinline__ double a16(double v) {  // the 8-lane butterfly, then the row's halves
    v = grp_sum(v);
    return v + dpp_move<0x140>(v);
}
__device__ __forceinline__ Dl da16(Dl a) { return {a16(a.v), a16(a.d)}; }
__device__ __forceinline__ DV3 da16_3(DV3 a) { return {da16(a.x), da16(a.y), da16(a.z)}; }
__device__ __forceinline__ void adj_grp_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__global__ void __launch_bounds__(kBGrp * kBGrpPerBlock) k_adj_surface_big(AdjArgs A) {
    __shared__ BPt spt[kBGrpPerBlock][kBPts];
    const DevMesh &m = A.m;
    const int g = threadIdx.x / kBGrp, lf = threadIdx.x % kBGrp;
    BPt *P = spt[g];
    const int npair = A.w.counters[kAdjDirsBig];
    const size_t nc = m.n_cells;
    const DV3 Z = dv(D3{0, 0, 0});
    for (int idx = blockIdx.x * kBGrpPerBlock + g; idx < npair; idx += gridDim.x * kBGrpPerBlock) {
        const int64_t pr = A.w.dlist_big[idx];
        const int c = (int)(pr >> 6), dir = (int)(pr & 63);
        const int bi = m.cbig[c];
        const double aP = A.alpha[c];
        const double V6 = 6.0 * m.vol[c];
        const double dtc = cell_dt(m, A.dt_dom, A.dt, c);
        const int v0 = m.bv_ptr[bi], nv = m.bv_ptr[bi + 1] - v0;
        D3 xp[2];
        double ap[2];
        D3 xs{0, 0, 0};
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int i = lf + kBGrp * h;
            xp[h] = D3{0, 0, 0};
            ap[h] = 0.0;
            if (i < nv) {
                const double *q = m.bv_xyz + 3 * (size_t)(v0 + i);
                xp[h] = D3{q[0], q[1], q[2]};
                const int k = m.bv_cls[v0 + i];
                double av = 0.0;
                for (int e = m.st_ptr[k]; e < m.st_ptr[k + 1]; ++e) av += m.st_w[e] * A.alpha[m.st_cell[e]];
                ap[h] = av;
                xs = xs + xp[h];
            }
        }
        const D3 xm = (1.0 / nv) * D3{a16(xs.x), a16(xs.y), a16(xs.z)};
        adj_grp_sync();  // the previous pair's reads of P are done
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int i = lf + kBGrp * h;
            if (i < nv) P[i] = BPt{xp[h].x - xm.x, xp[h].y - xm.y, xp[h].z - xm.z, ap[h]};
        }
        adj_grp_sync();
        const double iso = A.iso[c];
        const Dl isod{iso, dir == kBigIsoDir ? 1.0 : 0.0};
        // this lane's face: its loop of local points (outward), planarity, flux face
        const int f0 = m.bf_ptr[bi], nf = m.bf_ptr[bi + 1] - f0;
        const bool face = lf < nf;
        const int lb = face ? m.bl_ptr[f0 + lf] : 0;
        const int ln = face ? m.bl_ptr[f0 + lf + 1] - lb : 0;
        const bool planar = face && m.bf_planar[f0 + lf];
        auto loc = [&](int pos) { return m.bl_vtx[lb + pos]; };
        auto dpt = [&](int l) { return DV3{dc(P[l].x), dc(P[l].y), dc(P[l].z)}; };
        auto dval = [&](int l) { return Dl{P[l].a, l == dir ? 1.0 : 0.0}; };
        // cut point of the edge between local points l1 and l2, exactly one of them wet: from the
        // wet end, as the forward computes it
        auto cut = [&](int l1, int l2, bool w1) {
            const int lw = w1 ? l1 : l2, ld = w1 ? l2 : l1;
            const Dl lam = (isod - dval(lw)) / (dval(ld) - dval(lw));
            return dpt(lw) + lam * (dpt(ld) - dpt(lw));
        };
        // the face's share of six times the sub-volume and of the isoface sums (wet iff a > iso)
        DV3 C = Z, pacc = Z, psum = Z, lastexit = Z, first_entry = Z, cseg = Z, oacc = Z;
        Dl pl = dc(0.0), oL = dc(0.0);
        int cnt = 0;
        bool have_exit = false, pend = false;
        auto iso_edge = [&](DV3 s0, DV3 s1) {
            const Dl l = dnorm(s1 - s0);
            cseg = cseg + dcross(s0, s1);
            oacc = oacc + (0.5 * l) * (s0 + s1);
            oL = oL + l;
        };
        for (int i = 0; i < ln; ++i) {
            const int li = loc(i), lj = loc(i + 1 < ln ? i + 1 : 0);
            const bool wi = P[li].a > iso, wj = P[lj].a > iso;
            const DV3 xi = dpt(li), xj = dpt(lj);
            DV3 ct = Z;
            if (wi != wj) ct = cut(li, lj, wi);
            if (!wi && wj) {
                if (have_exit) iso_edge(ct, lastexit);
                else { pend = true; first_entry = ct; }
            }
            if (wi && !wj) { lastexit = ct; have_exit = true; }
            if (wi || wj) {
                const DV3 u = wi ? xi : ct, v = wj ? xj : ct;
                C = C + dcross(u, v);
                const Dl l = dnorm(v - u);
                pacc = pacc + (0.5 * l) * (u + v);
                pl = pl + l;
            }
            if (wi) psum = psum + xi;
            if (wi != wj) psum = psum + ct;
            cnt += (wi ? 1 : 0) + (wi != wj ? 1 : 0);
        }
        if (pend) iso_edge(first_entry, lastexit);
        C = C - cseg;  // the isoface edges close the wet loop, walked exit to entry
        Dl v6 = dc(0.0);
        if (cnt >= 3) {
            DV3 apx = dpt(loc(0));
            if (!planar) {
                const DV3 tot = pacc + oacc;
                const Dl tl = pl + oL;
                apx = tl.v > 0.0 ? dinv(tl) * tot : (1.0 / cnt) * psum;
            }
            v6 = ddot(apx, C);
        }
        const DV3 gcseg = da16_3(cseg), goacc = da16_3(oacc);
        const Dl goL = da16(oL);
        const DV3 o = goL.v > 0.0 ? dinv(goL) * goacc : Z;
        const Dl g0 = da16(v6) + ddot(o, gcseg);
        const Dl nrm = dnorm(gcseg);
        double contrib = 0.0;
        if (nrm.v > 0.0) {
            const DV3 nS = dinv(nrm) * gcseg;
            // the isoface centre: fan triangles (o, entry, preceding exit) weighted along n_S
            DV3 acc = Z;
            Dl ws = dc(0.0);
            DV3 le = Z, fe = Z;
            bool hx = false, pd = false;
            auto tri = [&](DV3 s0, DV3 s1) {
                const Dl wt = ddot(dcross(s0 - o, s1 - o), nS);
                acc = acc + wt * (o + s0 + s1);
                ws = ws + wt;
            };
            for (int i = 0; i < ln; ++i) {
                const int li = loc(i), lj = loc(i + 1 < ln ? i + 1 : 0);
                const bool wi = P[li].a > iso, wj = P[lj].a > iso;
                if (!wi && wj) {
                    const DV3 ct = cut(li, lj, false);
                    if (hx) tri(ct, le);
                    else { pd = true; fe = ct; }
                }
                if (wi && !wj) { le = cut(li, lj, true); hx = true; }
            }
            if (pd) tri(fe, le);
            acc = da16_3(acc);
            ws = da16(ws);
            const DV3 xS = dinv(3.0 * ws) * acc;
            const Dl un = A.U[c] * nS.x + A.U[nc + c] * nS.y + A.U[2 * nc + c] * nS.z;
            if (face) {
                const int32_t v = m.bf_face[f0 + lf];
                if (v != kEmpty) {
                    const int32_t fid = v >= 0 ? v : ~v;
                    const double ph = A.phi[fid];
                    const double out = v >= 0 ? ph : -ph;
                    if (out > 0.0) {
                        // the face fanned about its vertex mean, each triangle's swept fraction
                        D3 fm{0, 0, 0};
                        for (int i = 0; i < ln; ++i) {
                            const int l = loc(i);
                            fm = fm + D3{P[l].x, P[l].y, P[l].z};
                        }
                        fm = (1.0 / ln) * fm;
                        const Dl dap = ddot(dv(fm) - xS, nS);
                        Dl accI = dc(0.0);
                        double Af = 0.0;
                        for (int i = 0; i < ln; ++i) {
                            const int li = loc(i), lj = loc(i + 1 < ln ? i + 1 : 0);
                            const D3 xi{P[li].x, P[li].y, P[li].z}, xj{P[lj].x, P[lj].y, P[lj].z};
                            const double Ai = 0.5 * norm3(cross(xi - fm, xj - fm));
                            accI = accI + Ai * dtri_sweep(dap, ddot(dv(xi) - xS, nS), ddot(dv(xj) - xS, nS), un, dtc);
                            Af += Ai;
                        }
                        contrib = A.w.vbar[fid] * (accI.d / Af);
                    }
                }
            }
        }
        const double gsum = a16(contrib);
        double *gb = A.w.gbig + (size_t)kAdjGBig * bi;
        const int slot = dir == kBigIsoDir ? kBigIsoDir : dir;
        if (lf == 0) {
            gb[slot] = g0.d;
            gb[kBigC + slot] = gsum;
        }
        if (dir == kBigIsoDir) {
            // at a jump of the sub-volume the isovalue is a vertex value and moves with it: the
            // lowest point at the isovalue
            const bool jump = fabs(g0.v - aP * V6) > 1e-9 * V6;
            const int base = __lane_id() & ~(kBGrp - 1);
            const uint32_t lo = (uint32_t)(__ballot(lf < nv && P[lf].a == iso) >> base) & 0xFFFFu;
            const uint32_t hi = (uint32_t)(__ballot(lf + kBGrp < nv && P[lf + kBGrp].a == iso) >> base) & 0xFFFFu;
            const uint32_t at = lo | (hi << 16);
            if (lf == 0) {
                gb[kBigJump] = jump ? (double)(at ? __ffs((int)at) - 1 : -1) : -2.0;
                gb[kBigV6] = V6;
            }
        }
        // zero rates for the unused point slots, so that the gathers may read any of them
        if (dir == kBigIsoDir && lf == 0)
            for (int v = nv; v < kBigIsoDir; ++v) gb[v] = gb[kBigC + v] = 0.0;
    }
}

__device__ __forceinline__ double adj_vertex_big(const double *gb, int v) {
    const double jump = gb[kBigJump], gx = gb[kBigIsoDir];
    double xdot;
    if (jump > -2.0) xdot = (double)v == jump ? 1.0 : 0.0;
    else xdot = gx != 0.0 ? -gb[v] / gx : 0.0;
    return gb[kBigC + v] + xdot * gb[kBigC + kBigIsoDir];
}
__device__ __forceinline__ double adj_alpha_big(const double *gb) {
    const double gx = gb[kBigIsoDir];
    const double xdot = gb[kBigJump] > -2.0 ? 0.0 : (gx != 0.0 ? gb[kBigV6] / gx : 0.0);
    return xdot * gb[kBigC + kBigIsoDir];
}

// Transpose of the vertex interpolation, as two gathers in a fixed order (no atomics, so the
// gradient is the same bits on every run): each point class sums the vertex adjoints of the
// reconstructed cells that share it, then each cell adds its classes' sums times its weight in
// their stencils.  A cell that shares a class twice (two of its vertices are periodic images of
// one point) appears twice in the class's stencil, with one weight per image; its vertices are
// summed at its first entry and each of its distinct classes is taken once.

// The sum of class k over its stencil, of fixed width kN (a mesh of rectangular hexahedra): whole stencils by
// 16-byte loads (a class's entries one by one ask for the same lines eight times over: 24.4 us, this 10.5, on
// 128x64x64 cells).  Their padding repeats the first entry.
template <int kN>
__device__ __forceinline__ double point_sum(const AdjArgs &A, int k) {
    const DevMesh &m = A.m;
    const int4 *cp = reinterpret_cast<const int4 *>(m.sten_cell + (size_t)kN * k);
    int32_t c[kN], kd[kN];
#pragma unroll
    for (int j = 0; j < kN; j += 4) {
        const int4 q = cp[j / 4];
        c[j] = q.x; c[j + 1] = q.y; c[j + 2] = q.z; c[j + 3] = q.w;
    }
#pragma unroll
    for (int j = 0; j < kN; ++j) kd[j] = A.kind[c[j]];
    double sum = 0.0;
#pragma unroll
    for (int j = 0; j < kN; ++j) {
        bool first = kd[j] == 1;
#pragma unroll
        for (int i = 0; i < j; ++i) first = first && c[i] != c[j];
        if (!first) continue;
        const int4 *p = reinterpret_cast<const int4 *>(m.cpt + 8 * (size_t)c[j]);
        const int4 lo = p[0], hi = p[1];
        const int32_t cls[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
        for (int v = 0; v < 8; ++v)
            if (cls[v] == k) sum += A.w.gbuf[(size_t)kAdjG * c[j] + v];
    }
    return sum;
}

__global__ void __launch_bounds__(256) k_adj_points(AdjArgs A) {
    const DevMesh &m = A.m;
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= m.n_classes) return;
    if (m.box == 1) {
        A.w.pbar[k] = m.sten_n == 4 ? point_sum<4>(A, k) : point_sum<8>(A, k);
        return;
    }
    const int e0 = m.st_ptr[k], e1 = m.st_ptr[k + 1];
    double sum = 0.0;
    // stencil entries eight at a time, their cells' kinds all in flight together; most classes
    // have no reconstructed cell, and those skip the rest
    for (int eb = e0; eb < e1; eb += 8) {
        int32_t sc[8], kd[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) sc[j] = eb + j < e1 ? m.st_cell[eb + j] : -1;
#pragma unroll
        for (int j = 0; j < 8; ++j) kd[j] = sc[j] >= 0 ? A.kind[sc[j]] : 0;
        for (int j = 0; j < 8; ++j) {
            if (kd[j] != 1) continue;
            const int32_t c = sc[j];
            bool first = true;
            for (int e2 = e0; e2 < eb + j; ++e2) first = first && m.st_cell[e2] != c;
            if (!first) continue;
            if (m.cbig && m.cbig[c] >= 0) {
                const int bi = m.cbig[c], v0 = m.bv_ptr[bi], nv = m.bv_ptr[bi + 1] - v0;
                for (int v = 0; v < nv; ++v)
                    if (m.bv_cls[v0 + v] == k) sum += adj_vertex_big(A.w.gbig + (size_t)kAdjGBig * bi, v);
                continue;
            }
#pragma unroll
            for (int v = 0; v < 8; ++v)
                if (m.cpt[8 * (size_t)c + v] == k) sum += A.w.gbuf[(size_t)kAdjG * c + v];
        }
    }
    A.w.pbar[k] = sum;
}

// acc plus cell c's weight times the adjoint in each of its classes' stencils of width kN; those of four
// classes in flight together (entry by entry the kernel took 18.0 us on 128x64x64 cells, this 10.0).
template <int kN>
__device__ __forceinline__ double cell_sum(const DevMesh &m, int c, const int32_t (&cls)[8], const double (&pb)[8], double acc) {
#pragma unroll
    for (int v0 = 0; v0 < 8; v0 += 4) {
        uint32_t hit[4];
        double w[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int4 *cp = reinterpret_cast<const int4 *>(m.sten_cell + (size_t)kN * cls[v0 + v]);
            hit[v] = 0;
#pragma unroll
            for (int j = 0; j < kN; j += 4) {
                const int4 q = cp[j / 4];
                hit[v] |= ((q.x == c ? 1u : 0u) | (q.y == c ? 2u : 0u) | (q.z == c ? 4u : 0u) | (q.w == c ? 8u : 0u)) << j;
            }
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) w[v] = m.sten_w[(size_t)kN * cls[v0 + v] + (hit[v] ? __ffs(hit[v]) - 1 : 0)];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            if (pb[v0 + v] == 0.0) continue;
            if (hit[v]) acc += w[v] * pb[v0 + v];
            for (uint32_t h = hit[v] & (hit[v] - 1); h; h &= h - 1)  // a class the cell shares twice, or padding
                acc += m.sten_w[(size_t)kN * cls[v0 + v] + __ffs(h) - 1] * pb[v0 + v];
        }
    }
    return acc;
}

__global__ void __launch_bounds__(256) k_adj_cells(AdjArgs A) {
    const DevMesh &m = A.m;
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    // nothing reads the counters after the surface kernels: leave them zero for the next call
    if (blockIdx.x == 0 && threadIdx.x < kAdjNum) A.w.counters[threadIdx.x] = 0;
    if (c >= m.n_cells) return;
    double acc = A.abar[c];
    if (m.cbig && m.cbig[c] >= 0) {
        // a general polyhedron: the distinct classes of all its points
        const int bi = m.cbig[c], v0 = m.bv_ptr[bi], nv = m.bv_ptr[bi + 1] - v0;
        if (A.kind[c] == 1) acc += adj_alpha_big(A.w.gbig + (size_t)kAdjGBig * bi);
        for (int v = 0; v < nv; ++v) {
            const int32_t k = m.bv_cls[v0 + v];
            bool seen = false;
            for (int u = 0; u < v; ++u) seen = seen || m.bv_cls[v0 + u] == k;
            const double pbk = A.w.pbar[k];
            if (seen || pbk == 0.0) continue;
            for (int e = m.st_ptr[k]; e < m.st_ptr[k + 1]; ++e)
                if (m.st_cell[e] == c) acc += m.st_w[e] * pbk;
        }
        A.abar[c] = acc;
        return;
    }
    if (A.kind[c] == 1) acc += A.w.gbuf[(size_t)kAdjG * c + 8];
    const int4 *cp = reinterpret_cast<const int4 *>(m.cpt + 8 * (size_t)c);
    const int4 lo = cp[0], hi = cp[1];
    const int32_t cls[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
    double pb[8];
#pragma unroll
    for (int v = 0; v < 8; ++v) pb[v] = A.w.pbar[cls[v]];  // all eight in flight together
    bool any = false;
#pragma unroll
    for (int v = 0; v < 8; ++v) {
#pragma unroll
        for (int u = 0; u < v; ++u)
            if (cls[u] == cls[v]) pb[v] = 0.0;  // each distinct class once
        any = any || pb[v] != 0.0;
    }
    if (any) {
        if (m.box == 1) {
            acc = m.sten_n == 4 ? cell_sum<4>(m, c, cls, pb, acc) : cell_sum<8>(m, c, cls, pb, acc);
        } else {
#pragma unroll
            for (int v = 0; v < 8; ++v) {
                if (pb[v] == 0.0) continue;
                for (int e = m.st_ptr[cls[v]]; e < m.st_ptr[cls[v] + 1]; ++e)
                    if (m.st_cell[e] == c) acc += m.st_w[e] * pb[v];
            }
        }
    }
    A.abar[c] = acc;
}


template <int W>
hipError_t launch_adj_w(const AdjArgs &a, hipStream_t s) {
    static_assert(W <= 16, "the bounding tape's flags hold 16 slots");
    const int n = a.m.n_cells;
    const int g = (n + 255) / 256;
    const int gb = std::max(1, std::min(g, (int)kAdjBoundBlocks));
    hipLaunchKernelGGL(k_adj_prep<W>, dim3(g), dim3(256), 0, s, a);
    const int grid = std::min(a.n_iter, n <= kBoundGroupCells ? 0 : 1);  // sweeps over the whole grid
    for (int it = 0; it < grid; ++it) hipLaunchKernelGGL(k_adj_sweep<W>, dim3(gb), dim3(256), 0, s, a, it);
    const int gt = adj_group_threads(W);
    if (grid < a.n_iter)
        hipLaunchKernelGGL(k_adj_group<W>, dim3(bound_groups(n, W, gt)), dim3(gt), 0, s, a, grid);
    for (int it = grid - 1; it >= 0; --it) {
        hipLaunchKernelGGL(k_adj_unsweep_apply<W>, dim3(gb), dim3(256), 0, s, a, it);
        hipLaunchKernelGGL(k_adj_unsweep_correct<W>, dim3(gb), dim3(256), 0, s, a, it);
    }
    hipLaunchKernelGGL(k_adj_faces<W>, dim3(g), dim3(256), 0, s, a);
    const int gs = std::max(1, std::min(4096, (int)(((long)n * kLanes + 63) / 64)));
    hipLaunchKernelGGL(k_adj_surface, dim3(gs), dim3(64), 0, s, a);
    if (a.m.cbig) {
        const int gb = std::max(1, std::min(1024, (int)((33L * a.w.big_cap + kBGrpPerBlock - 1) / kBGrpPerBlock)));
        hipLaunchKernelGGL(k_adj_surface_big, dim3(gb), dim3(kBGrp * kBGrpPerBlock), 0, s, a);
    }
    hipLaunchKernelGGL(k_adj_points, dim3((a.m.n_classes + 255) / 256), dim3(256), 0, s, a);
    hipLaunchKernelGGL(k_adj_cells, dim3(g), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_adjoint(const DevMesh &m, const Params &p, const StepArgs &a, const AdjInputs &in, const AdjWork &w,
                          hipStream_t s) {
    if (p.n_bound_iter > kAdjMaxSweeps) return hipErrorInvalidValue;
    // phi_bar starts at zero in k_adj_prep (faces that carry no flux keep it); the counters are
    // zero from the workspace's allocation and left zero by k_adj_cells at the end of every call
    AdjArgs A{m, a.alpha, a.phi, a.U, a.dt, a.dt_dom, p.eps_surf, p.bound_tol, p.clip, p.n_bound_iter,
              in.vert_alpha, in.kind, in.iso, in.dV, in.raw, in.abar_new, in.abar, in.phibar, w};
    switch (m.W) {  // the slot widths of the step's update (polyhedra pad theirs to 8, 12 or 16)
        case 1: return launch_adj_w<1>(A, s);
        case 2: return launch_adj_w<2>(A, s);
        case 3: return launch_adj_w<3>(A, s);
        case 4: return launch_adj_w<4>(A, s);
        case 5: return launch_adj_w<5>(A, s);
        case 6: return launch_adj_w<6>(A, s);
        case 8: return launch_adj_w<8>(A, s);
        case 12: return launch_adj_w<12>(A, s);
        case 16: return launch_adj_w<16>(A, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace isoadv
