// Device helpers shared by the forward and adjoint kernels of the isoAdvector step (gfx950,
// wave64, FP64): small vectors, the canonical hexahedron's edge tables, a lane's face data, cut
// points, group reductions over the eight lanes of an interface cell, and list appends.
#pragma once

#include <hip/hip_runtime.h>

#include "internal.h"

namespace isoadv {
namespace {

constexpr int kLanes = 8;  // lanes per interface cell

struct D3 {
    double x, y, z;
};
__device__ __forceinline__ D3 operator+(D3 a, D3 b) { return {a.x + b.x, a.y + b.y, a.z + b.z}; }
__device__ __forceinline__ D3 operator-(D3 a, D3 b) { return {a.x - b.x, a.y - b.y, a.z - b.z}; }
__device__ __forceinline__ D3 operator*(double s, D3 a) { return {s * a.x, s * a.y, s * a.z}; }
__device__ __forceinline__ double dot(D3 a, D3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
__device__ __forceinline__ D3 cross(D3 a, D3 b) {
    return {a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x};
}
__device__ __forceinline__ double norm3(D3 a) { return sqrt(dot(a, a)); }
// component-wise select (a select of the whole struct can be lowered through memory)
__device__ __forceinline__ D3 sel3(bool c, D3 a, D3 b) { return D3{c ? a.x : b.x, c ? a.y : b.y, c ? a.z : b.z}; }

__device__ __forceinline__ bool interface_cell(double a, double eps) { return a > eps && a < 1.0 - eps; }

// Time step of cell c: the scalar one, or its ensemble member's (binary search over the members'
// cell offsets, a table of at most a few hundred bytes that stays in cache).
// the ensemble member holding cell c (0 for a single mesh)
__device__ __forceinline__ int cell_dom(const DevMesh &m, int c) {
    int lo = 0, hi = m.n_dom;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (m.dom_off[mid] <= c) lo = mid; else hi = mid;
    }
    return lo;
}

__device__ __forceinline__ double cell_dt(const DevMesh &m, const double *dt_dom, double dt, int c) {
    return m.n_dom <= 0 ? dt : dt_dom[cell_dom(m, c)];
}

// edges of the canonical hexahedron, and for each face loop position the edge to the next vertex

constexpr bool face_edges_consistent() {
    for (int k = 0; k < 6; ++k)
        for (int i = 0; i < 4; ++i) {
            const int p = kHexFace[k][i], q = kHexFace[k][(i + 1) & 3], e = kFaceEdge[k][i];
            if (!((kEdge[e][0] == p && kEdge[e][1] == q) || (kEdge[e][0] == q && kEdge[e][1] == p))) return false;
        }
    return true;
}
static_assert(face_edges_consistent(), "face/edge tables disagree");


// Work-groups are dispatched to the 8 XCDs round-robin (group b on XCD b mod 8), and each XCD has
// its own L2.  This bijection renumbers groups so that each XCD works through one contiguous
// range (consecutive logical groups, hence neighbouring cells and the faces and stencils they
// share, stay behind one L2).
constexpr int kXcds = 8;
__device__ __forceinline__ int xcd_block(int b, int nb) {
    const int x = b % kXcds, k = b / kXcds;
    const int q = nb / kXcds, r = nb % kXcds;
    return x * q + min(x, r) + k;
}

// Vertex loop of face lv (lanes 6 and 7 take face 0's) and, as bit i, whether loop position i runs
// along the canonical edge direction.
__device__ __forceinline__ int lane_face_loop(int lv, int *fv) {
    int fwd = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        fv[i] = kHexFace[0][i];
        int e = kFaceEdge[0][i];
#pragma unroll
        for (int k = 1; k < 6; ++k)
            if (lv == k) { fv[i] = kHexFace[k][i]; e = kFaceEdge[k][i]; }
        int first = kEdge[0][0];
#pragma unroll
        for (int t = 1; t < 12; ++t)
            if (e == t) first = kEdge[t][0];
        if (first == fv[i]) fwd |= 1 << i;
    }
    return fwd;
}

// ------------------------------------------------------------------------------------------ faces
// The eight lanes of an interface cell's group split every sub-volume evaluation by face: lane k
// (k < 6) owns canonical face k, its four vertices (relative to the cell's vertex mean), their
// values, and the reciprocal value difference along each of its edges.  Lanes 6 and 7 only help
// gathering vertex values.
struct FaceLane {
    D3 q[4];
    double aq[4];
    double inv[4];  // 1/(a_j - a_i) of the canonical edge (i, j) under loop position k
    int fwd;        // bit k: loop position k runs along the canonical edge direction
    bool planar;
    bool active;
};

// Cut point on the face edge from loop position i to i+1, measured from its wet end; both faces
// sharing the edge evaluate the same expression on the same operands, so they agree bitwise.
__device__ __forceinline__ D3 face_cut(const FaceLane &f, int i, double iso, bool wet_i) {
    const int j = (i + 1) & 3;
    const bool fwd = (f.fwd >> i) & 1;
    const D3 xw = sel3(wet_i, f.q[i], f.q[j]), xd = sel3(wet_i, f.q[j], f.q[i]);
    const double aw = wet_i ? f.aq[i] : f.aq[j];
    // wet end is the canonical edge's first vertex iff (wet_i == fwd)
    const double lam = (wet_i == fwd) ? (iso - aw) * f.inv[i] : (aw - iso) * f.inv[i];
    return xw + lam * (xd - xw);
}

// ------------------------------------------------------------------------------------------ lanes
// Reductions and broadcasts inside a group of 8 consecutive lanes (one interface cell).  The sum
// is a butterfly on DPP lane moves (swap neighbours, swap pairs inside a quad, mirror the two
// quads of the half-row): each step adds the same two partial sums in both partner lanes, so all
// lanes hold bitwise-equal results.  All 8 lanes of a group are active together (every branch
// around a reduction depends only on group-uniform values).
template <int Ctrl>
__device__ __forceinline__ double dpp_move(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_mov_dpp((int)b, Ctrl, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), Ctrl, 0xF, 0xF, true);
    return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}
constexpr int kDppSwap1 = 0xB1;       // quad_perm [1,0,3,2]
constexpr int kDppSwap2 = 0x4E;       // quad_perm [2,3,0,1]
constexpr int kDppHalfMirror = 0x141; // row_half_mirror: lane i <- lane 7-i within 8
__device__ __forceinline__ double grp_sum(double v) {
    v += dpp_move<kDppSwap1>(v);
    v += dpp_move<kDppSwap2>(v);
    v += dpp_move<kDppHalfMirror>(v);
    return v;
}
__device__ __forceinline__ D3 grp_sum3(D3 v) { return D3{grp_sum(v.x), grp_sum(v.y), grp_sum(v.z)}; }
__device__ __forceinline__ double grp_get(double v, int src) { return __shfl(v, src, 8); }

// The face of a slot, and a quantity of the face as seen from the slot's cell (its sign turned on
// the neighbour's side).
__device__ __forceinline__ int32_t face_of(int32_t v) { return v ^ (v >> 31); }
__device__ __forceinline__ double seen_from(int32_t v, double q) {
    return __hiloint2double(__double2hiint(q) ^ (int)(v & 0x80000000), __double2loint(q));
}

// The flux of face f and the velocity of cell c; with a second time level (outer iterations,
// Crank-Nicolson) their averages, formed as they are read.
template <bool kAvg>
__device__ __forceinline__ double flux_at(const double *phi, const double *phi1, int32_t f) {
    if constexpr (kAvg) return 0.5 * (phi[f] + phi1[f]);
    else return phi[f];
}
__device__ __forceinline__ D3 vel_at(const double *U, const double *U1, int32_t c, size_t n) {
    if (U1) return D3{0.5 * (U[c] + U1[c]), 0.5 * (U[n + c] + U1[n + c]), 0.5 * (U[2 * n + c] + U1[2 * n + c])};
    return D3{U[c], U[n + c], U[2 * n + c]};
}

// Append `count` entries per lane to a device-wide list: one atomic per wave.  Returns the index of
// this lane's first entry.  Every active lane of the wave must call it (count may be 0).
__device__ __forceinline__ int wave_append(int count, int32_t *counter) {
    // the active lanes are a prefix of the wave (a whole wave, or the last wave of a work-group
    // whose size is not a multiple of 64): the highest of them holds the total and takes the slots
    const int lane = __lane_id();
    const int top = 63 - __clzll((unsigned long long)__ballot(1));
    int incl = count;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(incl, o, 64);
        if (lane >= o) incl += y;
    }
    const int total = __shfl(incl, top, 64);
    int base = 0;
    if (lane == top && total > 0) base = atomicAdd(counter, total);
    base = __shfl(base, top, 64);
    return base + incl - count;
}

// The same for three counters (up to 2^20 elements of a wave each), their atomics in flight together.  A count
// of zero takes none: cells out of bounds often have nothing to correct, and where thousands of waves append,
// their atomics on one line are what bounds them (the update of 128x64x64 cells, a tenth of them out of bounds:
// 232 us with an atomic of each wave for each counter, 135 without those of zero; a thousandth: 27 and 20).  A lane
// for each counter, so that one instruction takes all three: a branch for each waits for the one before (that
// step 305 us, 275 so; calm steps of 30 to 45 us are 0.5 to 1 us shorter).
__device__ __forceinline__ int3 wave_append3(int3 count, int32_t *cx, int32_t *cy, int32_t *cz) {
    const int lane = __lane_id();
    const int top = 63 - __clzll((unsigned long long)__ballot(1));
    const uint64_t own = (uint64_t)count.x | (uint64_t)count.y << 20 | (uint64_t)count.z << 40;
    uint64_t incl = own;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint64_t y = __shfl_up((unsigned long long)incl, o, 64);
        if (lane >= o) incl += y;
    }
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)incl, top), hi = __builtin_amdgcn_readlane((uint32_t)(incl >> 32), top);
    const uint64_t all = (uint64_t)hi << 32 | lo;
    const int nx = (int)(all & 0xFFFFF), ny = (int)((all >> 20) & 0xFFFFF), nz = (int)(all >> 40);
    int x, y, z;
    if (top >= 2) {  // a lane for each counter: one instruction
        const int mine = lane == 0 ? nx : lane == 1 ? ny : nz;
        int base = 0;
        if (lane < 3 && mine) base = atomicAdd(lane == 0 ? cx : lane == 1 ? cy : cz, mine);
        x = __builtin_amdgcn_readlane(base, 0);
        y = __builtin_amdgcn_readlane(base, 1);
        z = __builtin_amdgcn_readlane(base, 2);
    } else {
        x = y = z = 0;
        if (lane == 0) {
            if (nx) x = atomicAdd(cx, nx);
            if (ny) y = atomicAdd(cy, ny);
            if (nz) z = atomicAdd(cz, nz);
        }
        x = __builtin_amdgcn_readlane(x, 0);
        y = __builtin_amdgcn_readlane(y, 0);
        z = __builtin_amdgcn_readlane(z, 0);
    }
    const uint64_t before = incl - own;
    return make_int3(x + (int)(before & 0xFFFFF), y + (int)((before >> 20) & 0xFFFFF), z + (int)(before >> 40));
}

// ------------------------------------------------------------------------------------------ teams
// A launch whose work-groups share a chain of phases, cut into tiles.  The tiles of the first phase are drawn by
// ticket; whoever holds the first ticket leads: it works through every tile that nobody else takes, waits only
// for tiles that a running group has taken, opens the next phase that is worth sharing for those who wait for
// one, and sends them away when what is left is for itself.  So nothing depends on how many groups run at a
// time, or on their order.  The last group to leave zeroes the words for the next launch.
//
// Groups on different XCDs see each other's stores by fences of device scope: a release by the leader before it
// opens a phase and by the taker after a tile, an acquire by the taker before one and by the leader after all.
struct Team {
    unsigned long long word;  // next tile (bits 0..31), tiles of the phase (32..61), kTeamOver; 0 in the first phase
    uint32_t done;            // tiles finished in all phases together
    uint32_t ticket;          // tiles of the first phase drawn
    uint32_t left;            // groups that have left
    int32_t arg[7];           // the phase, for the tiles' code
    int32_t cnt[2][2];        // (k_bound_group: two banks of list lengths)
};
static_assert(sizeof(Team) == 4 * kTeamWords, "the team's words");
constexpr unsigned long long kTeamOver = 1ull << 63, kTeamLead = 1ull << 62;

// Words that other groups of the launch read and write.
template <typename T>
__device__ __forceinline__ T team_load(const T *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void team_store(T *p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ T team_add(T *p, T v) {
    return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Tiles of a phase over n items, and the threads of a group that work on one: short items want many groups, each
// of few waves (by 1024, 512, 256 and 128 items a tile a step of 64x32x32 cells with 7.9 k of them out of bounds took
// 119, 107, 97 and 95 us).
__device__ __forceinline__ int team_tiles(int n) { return min((int)gridDim.x, max(8, n >> 7)); }
__device__ __forceinline__ int team_width(int n, int tiles) { return min((n / tiles + 64) & ~63, (int)blockDim.x); }

// Before a release by thread 0: every wave's stores have reached this XCD's L2.
__device__ __forceinline__ void team_sync() {
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
}

// Takes tiles, tile(i) with all threads of the group, until the phase has none left; the first phase has
// `tiles`.  True when the work is over; `lead` is set in the group that leads.
template <typename F>
__device__ __forceinline__ bool team_work(Team *t, int tiles, bool &lead, F tile) {
    __shared__ unsigned long long taken;
    for (;;) {
        if (threadIdx.x == 0) {
            // (a word read without a claim has no tile left: the tests below hold for both)
            unsigned long long w = team_load(&t->word);
            if (w == 0) {
                if (team_load(&t->ticket) < (uint32_t)tiles) {
                    const uint32_t i = team_add(&t->ticket, 1u);
                    w = (unsigned long long)tiles << 32 | i | (i == 0 ? kTeamLead : 0);
                }
            } else if (!(w & kTeamOver) && (uint32_t)w < (uint32_t)(w >> 32)) {
                w = team_add(&t->word, 1ull);
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            }
            taken = w;
        }
        __syncthreads();
        const unsigned long long w = taken;
        __syncthreads();
        if (w & kTeamOver) return true;
        if (w & kTeamLead) lead = true;
        if ((uint32_t)w >= ((uint32_t)(w >> 32) & 0x3fffffffu)) return false;
        tile((int)(uint32_t)w);
        team_sync();
        if (threadIdx.x == 0) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            team_add(&t->done, 1u);
        }
    }
}

// The leader waits until `tiles` tiles in all are done; everybody's stores in them are seen afterwards.
__device__ __forceinline__ void team_close(Team *t, uint32_t tiles) {
    if (threadIdx.x == 0) {
        while (team_load(&t->done) != tiles) __builtin_amdgcn_s_sleep(1);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    __syncthreads();
}

// The leader opens a phase.  Its stores before, thread 0's to t->arg among them, are seen by whoever takes a tile.
__device__ __forceinline__ void team_open(Team *t, int tiles) {
    team_sync();
    if (threadIdx.x == 0) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        team_store(&t->word, (unsigned long long)tiles << 32);
    }
}

// The leader sends the others away.
__device__ __forceinline__ void team_dismiss(Team *t) {
    if (threadIdx.x == 0) team_store(&t->word, kTeamOver);
}

// The end of every group of the launch, the leader's after all its work.  True (thread 0 only) in the group that
// leaves last: no other group reads or writes a word of the team any more, and all of them are zero again.
__device__ __forceinline__ bool team_leave(Team *t) {
    team_sync();
    if (threadIdx.x != 0 || team_add(&t->left, 1u) != gridDim.x - 1) return false;
    uint32_t *words = reinterpret_cast<uint32_t *>(t);
    for (int i = 0; i < kTeamWords; ++i) team_store(words + i, 0u);
    return true;
}

}  // namespace
// ------------------------------------------------------------------------------------------ sweep
// Integral over s in [0, dt] of the submerged fraction of a triangle with signed distances
// d0..d2 from the isoface plane moving with normal speed un: the fraction at time s is
// G(un*s), G the area distribution of d over the triangle (a triangular distribution).
// [0, dt] is split where un*s crosses a vertex distance; on each piece G(un*s) is a quadratic
// in s, integrated exactly by Simpson's rule on the branch picked at the piece's midpoint.
__device__ __forceinline__ double tri_piece(int br, double z, double e1, double e2, double e3, double r31,
                                            double r21, double r32) {
    if (br == 0) return 0.0;
    if (br == 3) return 1.0;
    if (br == 1) {
        const double u = z - e1;
        return (u * r31) * (u * r21);
    }
    const double u = e3 - z;
    return 1.0 - (u * r31) * (u * r32);
}

__device__ __forceinline__ double tri_sweep(double d0, double d1, double d2, double un, double dt) {
    const double e1 = fmin(d0, fmin(d1, d2)), e3 = fmax(d0, fmax(d1, d2));
    const double e2 = fmax(fmin(d0, d1), fmin(fmax(d0, d1), d2));
    const double r31 = e3 > e1 ? 1.0 / (e3 - e1) : 0.0;
    const double r21 = e2 > e1 ? 1.0 / (e2 - e1) : 0.0;
    const double r32 = e3 > e2 ? 1.0 / (e3 - e2) : 0.0;
    auto branch = [&](double z) { return z < e1 ? 0 : (z < e2 ? 1 : (z < e3 ? 2 : 3)); };
    if (un == 0.0) return dt * tri_piece(branch(0.0), 0.0, e1, e2, e3, r31, r21, r32);
    const double inv = 1.0 / un;
    double s1 = e1 * inv, s2 = e2 * inv, s3 = e3 * inv;
    if (un < 0.0) {  // breakpoints in increasing time
        const double t = s1;
        s1 = s3;
        s3 = t;
    }
    const double bk[3] = {s1, s2, s3};
    double I = 0.0, a0 = 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const double a1 = k < 3 ? fmin(fmax(bk[k], 0.0), dt) : dt;
        if (a1 > a0) {
            const double m = 0.5 * (a0 + a1);
            const int br = branch(un * m);
            const double fa = tri_piece(br, un * a0, e1, e2, e3, r31, r21, r32);
            const double fm = tri_piece(br, un * m, e1, e2, e3, r31, r21, r32);
            const double fb = tri_piece(br, un * a1, e1, e2, e3, r31, r21, r32);
            I += (a1 - a0) * (fa + 4.0 * fm + fb) * (1.0 / 6.0);
            a0 = a1;
        }
    }
    return I;
}

}  // namespace isoadv
