// Device-side ray walk shared by the single-scene and batched samplers:
// dense-grid voxel DDA (the plain method) and VDB + hierarchical DDA
// (Sec. 2.3, Sec. 3), each in the loop structure of Alg. 1 ("DDA branch")
// or Alg. 2 ("DDA skip") of the supplementary material.
//
// One ray per lane.  A ray is split into segments owned by one cascade level
// each (finest level wins, Sec. 3); within a segment a cursor walks cells in
// ray order -- voxels for the dense grid; root tiles, internal-node tiles or
// leaf voxels for the VDB tree -- and the driver turns maximal runs of
// occupied cells into parameter intervals (lo, hi].  A visitor converts an
// interval into its lattice points: the count pass adds their number and
// keeps the runs, the traversal fill writes the samples.
#pragma once
#pragma clang fp contract(off)

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "geometry.hpp"
#include "internal.hpp"
#include "scan.hpp"

namespace ogv {

constexpr int kBlock = 256;

// ------------------------------------------------------------------ cursors

// One moving axis as a cursor steps along it, in "walk order": the voxel
// coordinate w rises by one per voxel crossed -- w = v for d > 0, w = ~v for
// d < 0, so blocks of 2^k voxels stay aligned in w -- and the plane a step out
// of w crosses is p = w + 1, crossed at
//   T(p) = fl(fl(fl(B + fl(p * hs)) - o) * r),   hs = h or -h,
// which is the plane crossing of the definition bit for bit (a sign moved
// through a product changes no rounding).  T never decreases along the ray.
// An axis that does not move has hs = 0, o = -(largest float), r = 1: every T is
// the largest float, which no parameter of a walk passes, with no test on any step;
// its `per` is such that a relocation's estimate (below) is sure and keeps the
// voxel.  (Beside box coordinates of 2^100 and more, which that T would feel, o is
// -inf and T +inf.)
struct WalkAxis {
    float B, hs, o, r;
    float per;      // approximate voxels per unit of parameter, for relocation
    int32_t flip;   // v = w ^ flip

    __device__ __forceinline__ float T(float p) const {
        return __fmul_rn(__fsub_rn(__fadd_rn(B, __fmul_rn(p, hs)), o), r);
    }
    __device__ __forceinline__ float T(int p) const { return T((float)p); }
};

// Axis a of level `lev` for a ray: plane geometry from the level's table
// (B, h = fl((A-B)/R)), origin and direction component and its correctly
// rounded reciprocal.  d == 0 and an infinite 1/d do not move.
__device__ __forceinline__ bool axis_moves(float d, float r) { return d != 0.0f && !__builtin_isinf(r); }

__device__ __forceinline__ WalkAxis walk_axis(const float *geom, int lev, int a, float o, float d, float r) {
    const float B = geom[12 * lev + a], h = geom[12 * lev + 3 + a];
    const bool moves = axis_moves(d, r);
    WalkAxis x;
    x.B = B;
    x.hs = moves ? (d > 0.0f ? h : -h) : 0.0f;
    x.o = moves ? o : fabsf(B) < 0x1p100f ? -0x1.fffffep127f : -__builtin_huge_valf();
    x.r = moves ? r : 1.0f;
    x.per = moves ? __builtin_amdgcn_rcpf(x.hs * x.r) : 65535.5f * 0x1p-128f;
    x.flip = moves && d < 0.0f ? -1 : 0;
    return x;
}

// Relocation after a step out of a cell larger than a voxel: the walk-order
// voxel of each axis that holds the parameters just after t, the largest e in
// [w, p-1] with T(e) <= t (w itself when w >= p), for a ray known to be in
// voxels w .. p-1 then (T(w) <= t <= T(p) = Tp).
//
// With real arithmetic that is p - ceil(q), q = (Tp - t) / (h |r|) voxels
// back from p.  Rounding moves a crossing by less than
// |r| 2^-24 (6.1 M + 3.1 |o|), M the largest plane coordinate, so two of them
// move q by less than 2^-20 (M + |o|) / h; computing q adds a relative 2^-21
// of at most 2^8 voxels.  Where q is further than `slack` (twice both bounds)
// from an integer, the estimate is the answer; elsewhere, one time in about
// a thousand, exact comparisons settle it, as they do for a NaN or infinite
// q.  An axis that does not move has q = 65535.5 at small t and half of it at
// t = 2^127, which keeps w (walks that go beyond are settled exactly).  Ten instructions an axis, where a binary search over eight voxels takes
// about thirty.
__device__ __forceinline__ float relocate_slack(const float *geom, int lev, int R, const float o[3], float tmax) {
    float s = tmax > 0x1p127f ? __builtin_huge_valf() : 0.0f;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float B = geom[12 * lev + a], h = geom[12 * lev + 3 + a];
        s = fmaxf(s, (fmaxf(fabsf(B), fabsf(B + (float)R * h)) + fabsf(o[a])) * geom[12 * lev + 6 + a]);
    }
    return s * 0x1p-19f + 0x1p-12f;
}

struct Relocation {
    int e;
    bool sure;
};
__device__ __forceinline__ Relocation relocate_estimate(const WalkAxis &A, int w, int p, float Tp, float t,
                                                        float slack) {
    const float q = (Tp - t) * A.per;
    // an axis that stepped is at w = p: there is nothing to settle
    return {(int)fmaxf((float)p - ceilf(q), (float)w), fabsf(q - rintf(q)) > slack || w >= p};
}
__device__ __forceinline__ int relocate_exact(const WalkAxis &A, int e, int w, int p, float t) {
    e = max(min(e, p - 1), w);
    while (e > w && A.T(e) > t) --e;
    while (e + 1 < p && A.T(e + 1) <= t) ++e;
    return e;
}
__device__ __forceinline__ void relocate(const WalkAxis &A0, const WalkAxis &A1, const WalkAxis &A2, int &w0, int &w1,
                                         int &w2, int p0, int p1, int p2, float t0, float t1, float t2, float t,
                                         float slack) {
    const Relocation a0 = relocate_estimate(A0, w0, p0, t0, t, slack);
    const Relocation a1 = relocate_estimate(A1, w1, p1, t1, t, slack);
    const Relocation a2 = relocate_estimate(A2, w2, p2, t2, t, slack);
    int e0 = a0.e, e1 = a1.e, e2 = a2.e;
    if (!(a0.sure & a1.sure & a2.sure)) {
        e0 = relocate_exact(A0, e0, w0, p0, t);
        e1 = relocate_exact(A1, e1, w1, p1, t);
        e2 = relocate_exact(A2, e2, w2, p2, t);
    }
    w0 = e0;
    w1 = e1;
    w2 = e2;
}

// The cursors share one step: exit() gives the parameter hi at which the ray
// leaves the current cell -- the smallest of the three axes' crossings, all
// computed on every step -- and advance(hi) moves every axis whose crossing
// is hi across its plane.  Computing all three and selecting costs fewer
// issue slots than one branch per axis, of which a wave runs each in turn
// because its lanes step along different axes.  Axes that tie step together:
// the cell between them would hold (hi, hi], no parameter at all.  A walk
// needs no test for leaving the grid: it ends when hi reaches the segment's
// end b, which is at most the first crossing of a last plane, and crossings
// never decrease, so a plane crossed at hi < b is not a last one.

// Dense bitfield: every cell is a voxel; one bit lookup per voxel.  The bit
// read for the new voxel is tested in the next step, after that step's
// crossings, so its latency overlaps them.
struct DenseCursor {
    const uint32_t *bits;   // word holding the level's first bits
    WalkAxis A0, A1, A2;
    float p0, p1, p2;       // next plane per axis, as a float (exact: at most 2^10)
    float t0, t1, t2;       // its crossing
    int32_t s0, s1, s2;     // bit-index change of a step along each axis
    uint32_t idx;           // bit index of the current voxel
    uint32_t word;          // its word

    // by a 32-bit byte offset from a uniform base (a level has at most 2^30 bits)
    __device__ __forceinline__ void fetch() {
        word = *reinterpret_cast<const uint32_t *>(reinterpret_cast<const char *>(bits) + ((idx >> 5) << 2));
    }
    __device__ __forceinline__ void start(const uint32_t *all, uint64_t level_base, int R, int w0, int w1, int w2) {
        bits = all + (level_base >> 5);
        const int v0 = w0 ^ A0.flip, v1 = w1 ^ A1.flip, v2 = w2 ^ A2.flip;
        idx = (uint32_t)(level_base & 31) + ((uint32_t)v0 * (uint32_t)R + (uint32_t)v1) * (uint32_t)R + (uint32_t)v2;
        s0 = ((R * R) ^ A0.flip) - A0.flip;
        s1 = (R ^ A1.flip) - A1.flip;
        s2 = 1 | A2.flip;
        p0 = (float)(w0 + 1);
        p1 = (float)(w1 + 1);
        p2 = (float)(w2 + 1);
        fetch();
    }
    __device__ __forceinline__ uint32_t occupied() const { return (word >> (idx & 31)) & 1u; }
    __device__ __forceinline__ float exit() {
        t0 = A0.T(p0);
        t1 = A1.T(p1);
        t2 = A2.T(p2);
        return fminf(fminf(t0, t1), t2);
    }
    __device__ __forceinline__ void advance(float hi) {
        const bool c0 = t0 <= hi, c1 = t1 <= hi, c2 = t2 <= hi;
        p0 += c0 ? 1.0f : 0.0f;
        p1 += c1 ? 1.0f : 0.0f;
        p2 += c2 ? 1.0f : 0.0f;
        idx += (uint32_t)(c0 ? s0 : 0) + (uint32_t)(c1 ? s1 : 0) + (uint32_t)(c2 ? s2 : 0);
        fetch();
    }
};

// The parts of a VDB tree a walk reads: the root table and the nodes' slot
// tables (staged in LDS when they fit), and the leaves (global memory).
struct Tree {
    const int32_t *root;
    const int32_t *slot;
    const uint64_t *leaves;
    const uint64_t *sub;   // [leaves]: uniform 4^3 sub-blocks
    int ilog2, S, NR;
};

__host__ __device__ inline size_t tree_lds_bytes(int L, int NR, int S) {
    const size_t n_root = (size_t)L * NR * NR * NR;
    return n_root * 4 + n_root * (size_t)S * S * S * 4;
}

// Copies n4 >= 1 16-byte words from global memory to LDS.  A thread issues
// the loads of a batch together and only then stores them, so the block waits
// for one memory round trip per batch rather than one per word.  Indices past
// the end are clamped to the last word, which such lanes load and store again
// with its own value: no branch lets the compiler sink a load to its store.
__device__ __forceinline__ void stage_to_lds(int4 *dst, const int4 *__restrict__ src, int n4) {
    constexpr int kBatch = 4;
    const int nt = (int)blockDim.x, t = (int)threadIdx.x;
    for (int base = 0; base < n4; base += kBatch * nt) {
        int4 r[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) r[u] = src[min(base + u * nt + t, n4 - 1)];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) dst[min(base + u * nt + t, n4 - 1)] = r[u];
    }
}

// The tree's view with its slot and root tables at smem (slot table first,
// then the root table: tree_lds_bytes), as stage_tree leaves them.  Node
// slots exist for every root cell (the worst case the build sizes for).
__device__ __forceinline__ Tree tree_in_lds(const GridView &g, uint32_t *smem) {
    Tree t;
    t.ilog2 = g.ilog2;
    t.S = g.S;
    t.NR = g.NR;
    t.leaves = g.leaves;
    t.sub = g.sub;
    const int ns = g.L * g.NR * g.NR * g.NR * g.S * g.S * g.S;
    t.slot = (const int32_t *)smem;
    t.root = (const int32_t *)smem + ns;
    return t;
}

// Copies the slot and root tables to smem.  Every thread of the block must
// call this (it synchronizes).  smem must be 16-byte aligned; the slot table
// is (the build aligns every table to 256 bytes, and a table holds S^3
// entries per root cell, a multiple of 4).
__device__ __forceinline__ void stage_tree(const GridView &g, uint32_t *smem) {
    const int n_root = g.L * g.NR * g.NR * g.NR;
    const int ns = n_root * g.S * g.S * g.S;
    int32_t *slot = (int32_t *)smem;
    int32_t *root = slot + ns;
    stage_to_lds(reinterpret_cast<int4 *>(slot), reinterpret_cast<const int4 *>(g.slot), ns >> 2);
    for (int i = threadIdx.x; i < n_root; i += blockDim.x) root[i] = g.root[i];
    __syncthreads();
}

// The tree a walk reads: its tables staged in LDS (kLds; every thread of the
// block must call this), or read from global memory.
template <bool kLds>
__device__ __forceinline__ Tree load_tree(const GridView &g, uint32_t *smem) {
    if (kLds) {
        stage_tree(g, smem);
        return tree_in_lds(g, smem);
    }
    Tree t;
    t.ilog2 = g.ilog2;
    t.S = g.S;
    t.NR = g.NR;
    t.leaves = g.leaves;
    t.sub = g.sub;
    t.root = g.root;
    t.slot = g.slot;
    return t;
}

// VDB tree: the current cell is the largest uniform cell holding the current
// voxel -- a root tile (D = 8*S voxels per axis), an internal-node tile
// (D = 8) or a leaf voxel (D = 1); with kSub, inside a leaf also a uniform
// 4^3 sub-block (D = 4: all its 64 voxels empty, or all occupied), so that
// the cells nest as aligned cubes of 8S, 8, 4 and 1 voxels a side and a step
// passes empty space by powers of two down to single voxels (Fig. 1).
//
// Cells are aligned in walk order too, so the exit plane of an axis is
// (w | (D-1)) + 1 whatever its direction.  While cells of one size or larger
// are crossed, the axes that do not step keep a voxel that may lie behind the
// ray but is in the same cell; only on the way into a finer cell are they
// relocated, exactly, at the exit parameter.  The 8^3 block entered is known
// before that (axes inside an 8^3 tile stay in its block), so the relocation
// follows the slot lookup and nothing is looked up twice.
//
// The slot table is read only when the block changes; the leaf's word is read
// for every leaf voxel and tested in the next step, after that step's
// crossings, so the walk waits for LDS but not for memory.
//
// kTiles = false walks the same tree one voxel per step (the paper's
// "VDB + DDA" rows, Tab. 1-2): a voxel inside a tile takes the tile's value
// and the walk moves on to the next voxel, so the tree only changes how
// occupancy is looked up, not which cells are visited.
template <bool kTiles, bool kSub = false>
struct VdbWalk {
    Tree t;
    int lev;
    int node;              // first slot of the current root cell's node, or the cell's tile value
    WalkAxis A0, A1, A2;
    int w0, w1, w2;        // voxel in walk order (inside the current cell)
    int p0, p1, p2;        // exit plane of the current cell
    float t0, t1, t2;      // its crossing
    float slack;           // relocate_slack
    int Dm1;               // current cell size in voxels, less one
    int lblk;              // 8^3 block last looked up (packed block coordinates), -1 if none
    int code;              // its table entry: leaf index, or a tile's value (kEmptyTile ...)
    uint32_t word, bit;    // current cell occupied: bit `bit` of `word`
    uint32_t lu4;          // kSub: uniform 4^3 sub-blocks of the leaf

    // table entries of tiles; even entries are occupied
    static constexpr int kEmptySlot = -1, kFullSlot = -2, kEmptyRoot = -3, kFullRoot = -4;

    __device__ __forceinline__ void set_node(int r) { node = r < 0 ? r - 2 : r << (3 * t.ilog2); }
    __device__ __forceinline__ void relocate_at(float hi) {
        relocate(A0, A1, A2, w0, w1, w2, p0, p1, p2, t0, t1, t2, hi, slack);
    }

    // The cell holding the current voxels, entered at hi from a cell of size
    // Dm1 + 1 (0: the voxels are exact), becomes current.
    __device__ __forceinline__ void lookup(float hi) {
        int v0 = w0 ^ A0.flip, v1 = w1 ^ A1.flip, v2 = w2 ^ A2.flip;
        const int blk = ((v0 >> 3) << 14) | ((v1 >> 3) << 7) | (v2 >> 3);
        if (blk != lblk) {
            lblk = blk;
            const int NR = t.NR, lg = t.ilog2;
            if (NR > 1) {
                const int sh = 3 + lg;
                set_node(t.root[((lev * NR + (v0 >> sh)) * NR + (v1 >> sh)) * NR + (v2 >> sh)]);
            }
            const int m = t.S - 1;
            const int s = (((((v0 >> 3) & m) << lg) | ((v1 >> 3) & m)) << lg) | ((v2 >> 3) & m);
            const int c = t.slot[max(node, 0) + s];
            code = node < 0 ? node : c;
            if (kSub && code >= 0) lu4 = (uint32_t)t.sub[code];
        }
        if (code >= 0) {
            if (kTiles && Dm1 != 0) {
                relocate_at(hi);
                v0 = w0 ^ A0.flip;
                v1 = w1 ^ A1.flip;
                v2 = w2 ^ A2.flip;
            }
            const uint32_t at = ((((uint32_t)v0 & 7) << 3 | ((uint32_t)v1 & 7)) << 3) | ((uint32_t)v2 & 7);
            // a 32-bit byte offset from a uniform base (at most 2^24 leaves of 64 bytes)
            word = *reinterpret_cast<const uint32_t *>(reinterpret_cast<const char *>(t.leaves) +
                                                       (((uint32_t)code << 6) | ((at >> 5) << 2)));
            bit = at & 31;
            Dm1 = 0;
            if (kSub) {
                // a uniform 4^3 sub-block takes the voxel's value and is the cell
                const int s4 = ((v0 & 4) | ((v1 & 4) >> 1) | ((v2 & 4) >> 2));
                Dm1 = ((lu4 >> s4) & 1u) != 0 ? 3 : 0;
            }
        } else {
            word = ~(uint32_t)code;   // bit 0: an even entry is occupied
            bit = 0;
            if (kTiles) Dm1 = code <= kEmptyRoot ? (8 << t.ilog2) - 1 : 7;
        }
    }

    __device__ __forceinline__ uint32_t occupied() const { return (word >> bit) & 1u; }

    __device__ __forceinline__ float exit() {
        p0 = (w0 | Dm1) + 1;
        p1 = (w1 | Dm1) + 1;
        p2 = (w2 | Dm1) + 1;
        t0 = A0.T(p0);
        t1 = A1.T(p1);
        t2 = A2.T(p2);
        return fminf(fminf(t0, t1), t2);
    }

    __device__ __forceinline__ void advance(float hi) {
        w0 = t0 <= hi ? p0 : w0;
        w1 = t1 <= hi ? p1 : w1;
        w2 = t2 <= hi ? p2 : w2;
        // out of a root tile the other axes may be in another block
        if (kTiles && Dm1 > 7) {
            relocate_at(hi);
            Dm1 = 0;
        }
        lookup(hi);
    }
};

// ------------------------------------------------------------------ driver

// Walks cells from the segment start a to its end b (or t_max) and reports
// maximal occupied runs (lo, hi] to the visitor.
// kSkip = false is Alg. 1 (every cell visited, branch on occupancy);
// kSkip = true is Alg. 2 (an inner loop passes all leading empty cells, then
// the occupied run is marched).
//
// A visitor that has no room for another run (vis.room) makes the loop of
// Alg. 1 stop on the cell that would close it; vis.make_room, outside the
// loop, empties its store, and the walk goes on from the same cell.
template <bool kSkip, class Cursor, class Vis, class Ctx>
__device__ __forceinline__ void drive(Cursor &c, float a, float b, float tmax, Vis &vis, const Ctx &ctx) {
    float lo = a;
    const float last = fminf(b, tmax);
    if (!kSkip) {
        uint32_t in_run = 0;
        float run_lo = a;
        while (true) {
            bool full = false;
            while (true) {
                const float hi = c.exit();
                const bool end = hi >= last;
                const uint32_t occ = c.occupied();
                if (occ > in_run) run_lo = lo;
                // a run closes at lo on an empty cell, or at this cell's end when the ray ends
                if ((in_run > occ) | (end & (occ != 0))) {
                    full = !vis.room(ctx);
                    if (full) break;
                    vis.run(ctx, run_lo, occ != 0 ? fminf(hi, b) : lo);
                }
                if (end) break;
                in_run = occ;
                c.advance(hi);
                lo = hi;
            }
            if (!full) return;
            vis.make_room(ctx);
        }
    } else {
        while (true) {
            bool end = false;
            while (!c.occupied()) {
                const float hi = c.exit();
                if (hi >= last) return;
                c.advance(hi);
                lo = hi;
            }
            float run_lo = lo, run_hi;
            while (true) {
                const float hi = c.exit();
                end = hi >= last;
                if (!end) c.advance(hi);
                run_hi = fminf(hi, b);
                lo = hi;
                if (end || !c.occupied()) break;
            }
            if (!vis.room(ctx)) vis.make_room(ctx);
            vis.run(ctx, run_lo, run_hi);
            if (end) return;
        }
    }
}

// ------------------------------------------------------------------ visitors

// Count pass: number of lattice points in each occupied run, and the runs
// themselves as lattice-index ranges [n0, n1) (adjacent ranges merged) for
// the expansion fill.  A ray keeps its first kMaxRuns runs in fixed slots;
// further runs go to chunks of kMaxRuns slots taken from a shared pool and
// chained (ray_next -> pool_next -> ...).  If the pool runs dry the ray is
// marked kRunsLost, listed, and the traversal fill writes it instead.
//
// During the walk a run is only recorded, as the bits of its parameter
// interval (lo, hi]; its lattice range is found once the walk has ended, in
// a loop over the ray's recorded runs that also merges adjacent ranges and
// rewrites them in place.  Lanes close runs at different steps, so doing the
// lattice arithmetic at the close would run it, masked, in most steps of a
// wave; after the walk the lanes of a wave do it together.  A ray whose runs
// are lost records into its fixed slots again and again; each time they are
// full the walk stops and they are counted and dropped (make_room).
constexpr int kMaxRuns = 16;
constexpr int32_t kRunsLost = 0x7fffffff;

struct RunPool {
    int2 *slots;          // [kMaxRuns][stride]: slot k of ray r at k * stride + r (reads of one slot coalesce)
    int64_t stride;       // rays the slot array is laid out for
    int32_t *ray_next;    // [rays]: first pool chunk of the ray, -1 if none
    int2 *chunks;         // [cap][kMaxRuns]
    int32_t *chunk_next;  // [cap]
    int32_t *head;        // chunks handed out so far
    int32_t cap;
    int32_t *lost;        // [rays]: rays marked kRunsLost, in no particular order
    int32_t *n_lost;      // their number
};

// Uniform context of the count pass.
struct CountCtx {
    Lattice lat;
    RunPool pool;
};

// Per-lane state of the count pass.
struct CountVis {
    int2 *at;             // where the next run is recorded
    int64_t ray;
    int32_t n;            // samples counted so far (of a lost ray before finish(), else 0)
    int32_t nr;           // runs recorded and not yet counted; after finish(), runs kept or kRunsLost
    int32_t chunk;        // last pool chunk taken, -1 if none, kDry once the pool has run dry
    static constexpr int32_t kDry = -2;

    __device__ __forceinline__ void begin_level(const GridView &, int, const float *, const float *) {}

    // room for one more run; takes the next pool chunk when the slots so far are used
    __device__ __forceinline__ bool room(const CountCtx &x) {
        const RunPool &pool = x.pool;
        if (nr == 0 || nr % kMaxRuns != 0) return true;
        if (chunk == kDry) return false;
        const int32_t c = atomicAdd(pool.head, 1);
        if (c >= pool.cap) return false;
        pool.chunk_next[c] = -1;
        if (nr == kMaxRuns) pool.ray_next[ray] = c;
        else pool.chunk_next[chunk] = c;
        chunk = c;
        at = pool.chunks + (int64_t)c * kMaxRuns;
        return true;
    }
    __device__ __forceinline__ void run(const CountCtx &x, float lo, float hi) {
        *at = make_int2(__float_as_int(lo), __float_as_int(hi));
        at += nr < kMaxRuns ? x.pool.stride : 1;
        ++nr;
    }
    // The pool is dry: the runs recorded so far are counted and dropped (the
    // fill re-walks this ray, so only its count is needed).
    __device__ __forceinline__ void make_room(const CountCtx &x) {
        walk_runs<false>(x);
        chunk = kDry;
        nr = 0;
        at = x.pool.slots + ray;
    }
    // lattice points of (lo, hi] up to t_max: [n0, n1), empty when n1 <= n0
    __device__ __forceinline__ static int2 lattice_range(const Lattice &lat, float lo, float hi) {
        return make_int2(lat.first_above(lo), lat.first_above(fminf(hi, lat.tmax)));
    }
    // Adds the lattice points of the nr recorded runs to n.  kKeep: the
    // ranges, merged where one ends at the next's start, are written back
    // over the recorded runs (the write index never passes the read index),
    // and nr becomes their number.
    template <bool kKeep>
    __device__ __forceinline__ void walk_runs(const CountCtx &x) {
        const RunPool &pool = x.pool;
        const int64_t stride = pool.stride;
        int2 *rp = pool.slots + ray, *wp = rp;
        int32_t rc = -1, wc = -1;        // pool chunks of the read and write positions
        int32_t c0 = 0, c1 = 0;          // merged range held back (c1 > c0 when held)
        int w = 0;
        const auto next = [&](int2 *&q, int32_t &c, int k) {   // q moves on to position k
            if (k < kMaxRuns) q += stride;
            else if (k % kMaxRuns != 0) q += 1;
            else {
                c = k == kMaxRuns ? pool.ray_next[ray] : pool.chunk_next[c];
                q = pool.chunks + (int64_t)c * kMaxRuns;
            }
        };
        const auto emit = [&]() {
            if (w > 0) next(wp, wc, w);
            *wp = make_int2(c0, c1);
            ++w;
        };
        for (int k = 0; k < nr; ++k) {
            if (k > 0) next(rp, rc, k);
            const int2 raw = *rp;
            const int2 q = lattice_range(x.lat, __int_as_float(raw.x), __int_as_float(raw.y));
            if (q.y <= q.x) continue;
            n += q.y - q.x;
            if (kKeep) {
                if (c1 > c0 && c1 == q.x) {
                    c1 = q.y;
                    continue;
                }
                if (c1 > c0) emit();
                c0 = q.x;
                c1 = q.y;
            }
        }
        if (kKeep) {
            if (c1 > c0) emit();
            nr = w;
        }
    }
    __device__ __forceinline__ void finish(const CountCtx &x) {
        if (chunk != kDry) {
            walk_runs<true>(x);
            return;
        }
        walk_runs<false>(x);
        nr = kRunsLost;
        x.pool.lost[atomicAdd(x.pool.n_lost, 1)] = (int32_t)ray;
    }
};

__device__ __forceinline__ CountVis make_count_vis(int64_t ray, const RunPool &pool) {
    CountVis v;
    v.at = pool.slots + ray;
    v.ray = ray;
    v.n = 0;
    v.nr = 0;
    v.chunk = -1;
    pool.ray_next[ray] = -1;
    return v;
}

// Uniform context of the traversal fill.
struct FillCtx {
    Lattice lat;
    int64_t capacity;
    int32_t *ray_ids;
    float *t0, *t1;
    int32_t *vox;         // written when kVox
    int R;
};

// Per-lane state of the traversal fill.
template <bool kVox>
struct FillVis {
    int64_t idx;
    int32_t ray;
    int lev;
    Axis A0, A1, A2;      // level geometry, for voxel ids only

    __device__ __forceinline__ void begin_level(const GridView &g, int l, const float *o, const float *d) {
        lev = l;
        if (kVox) {
            A0 = load_axis(g.geom, l, 0, g.R, o[0], d[0], __fdiv_rn(1.0f, d[0]));
            A1 = load_axis(g.geom, l, 1, g.R, o[1], d[1], __fdiv_rn(1.0f, d[1]));
            A2 = load_axis(g.geom, l, 2, g.R, o[2], d[2], __fdiv_rn(1.0f, d[2]));
        }
    }
    __device__ __forceinline__ bool room(const FillCtx &) { return true; }
    __device__ __forceinline__ void make_room(const FillCtx &) {}
    __device__ __forceinline__ static int vcoord(const Axis &A, float t) {
        return A.zero ? A.zero_voxel() : A.voxel(A.locate(t, false));
    }
    __device__ __forceinline__ void run(const FillCtx &x, float lo, float hi) {
        int n0 = x.lat.first_above(lo);
        int n1 = x.lat.first_above(fminf(hi, x.lat.tmax));
        float tn = x.lat.t(n0);
        for (int n = n0; n < n1; ++n) {
            float tnext = x.lat.t(n + 1);
            if (idx < x.capacity) {
                x.ray_ids[idx] = ray;
                x.t0[idx] = tn;
                x.t1[idx] = tnext;
                if (kVox) {
                    int i = vcoord(A0, tn), j = vcoord(A1, tn), k = vcoord(A2, tn);
                    x.vox[idx] = ((lev * x.R + i) * x.R + j) * x.R + k;
                }
            }
            ++idx;
            tn = tnext;
        }
    }
};

// Dense bitfield with chessboard distances (a traversal the paper discusses
// but does not evaluate, Sec. 2.3 and Fig. 1): in an empty voxel at distance d >= 2 from
// every occupied voxel, the whole cube of voxels within d - 1 of it is empty,
// so the ray leaves that cube in one step.  The cube's exit planes are the
// current voxel's plus d - 1 per axis; after the exit, the axes it did not
// leave through are relocated exactly at the exit parameter within the cube.
// Occupied voxels and empty ones at distance 1 are single cells, stepped as
// by the dense march.  A cube may reach past the grid, where T goes on.
struct DistCursor {
    const uint8_t *dist;   // the level's
    int R;
    WalkAxis A0, A1, A2;
    int w0, w1, w2;        // voxel in walk order
    int p0, p1, p2;        // exit plane of the current cell
    float t0, t1, t2;      // its crossing
    int d;                 // the current voxel's distance (0: occupied)
    float slack;           // relocate_slack

    __device__ __forceinline__ void lookup() {
        const uint32_t v0 = (uint32_t)(w0 ^ A0.flip), v1 = (uint32_t)(w1 ^ A1.flip), v2 = (uint32_t)(w2 ^ A2.flip);
        d = dist[(v0 * (uint32_t)R + v1) * (uint32_t)R + v2];
    }
    __device__ __forceinline__ uint32_t occupied() const { return d == 0 ? 1u : 0u; }
    __device__ __forceinline__ float exit() {
        const int n = max(d, 1);
        p0 = w0 + n;
        p1 = w1 + n;
        p2 = w2 + n;
        t0 = A0.T(p0);
        t1 = A1.T(p1);
        t2 = A2.T(p2);
        return fminf(fminf(t0, t1), t2);
    }
    __device__ __forceinline__ void advance(float hi) {
        w0 = t0 <= hi ? p0 : w0;
        w1 = t1 <= hi ? p1 : w1;
        w2 = t2 <= hi ? p2 : w2;
        if (d > 1) relocate(A0, A1, A2, w0, w1, w2, p0, p1, p2, t0, t1, t2, hi, slack);
        lookup();
    }
};

// ------------------------------------------------------------------ ray

struct Ray {
    float o[3], d[3], r[3];
};

__device__ __forceinline__ Ray make_ray(const float o[3], const float d[3]) {
    return Ray{{o[0], o[1], o[2]},
               {d[0], d[1], d[2]},
               {__fdiv_rn(1.0f, d[0]), __fdiv_rn(1.0f, d[1]), __fdiv_rn(1.0f, d[2])}};
}

// Traversals: 0 dense bitfield, 1 VDB tree with hierarchical steps, 2 dense
// bitfield with chessboard distances (GridView::kind 0, 1, 2), 3 the VDB
// tree walked one voxel per step and 4 the VDB tree with hierarchical steps
// that also pass uniform sub-blocks inside leaves (both on kind-1 grids).
template <int kGrid>
struct CursorOf {
    using type = DenseCursor;
};
template <>
struct CursorOf<1> {
    using type = VdbWalk<true>;
};
template <>
struct CursorOf<2> {
    using type = DistCursor;
};
template <>
struct CursorOf<3> {
    using type = VdbWalk<false>;
};
template <>
struct CursorOf<4> {
    using type = VdbWalk<true, true>;
};

// Traversals that read the VDB tree.
constexpr bool reads_tree(int kGrid) { return kGrid == 1 || kGrid == 3 || kGrid == 4; }

// One level as a ray meets it: its axes and the parameters (E, X] it holds.
struct RayLevel {
    WalkAxis A[3];
    float E, X;
};

// Entry and exit of the level box: the largest first and the smallest last
// crossing of the moving axes; the others must hold o inside (floor rule).
// False when the ray misses the level (or holds no parameter of it).
__device__ __forceinline__ bool meet_level(const GridView &g, int lev, const Ray &ray, RayLevel &m) {
    const float inf = __builtin_huge_valf();
    m.E = -inf;
    m.X = inf;
    bool in = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const WalkAxis A = walk_axis(g.geom, lev, a, ray.o[a], ray.d[a], ray.r[a]);
        const bool moves = axis_moves(ray.d[a], ray.r[a]);
        const int first = A.flip & -g.R;   // walk-order planes first .. first + R
        m.E = fmaxf(m.E, moves ? A.T(first) : -inf);
        m.X = fminf(m.X, A.T(first + g.R));
        const float P0 = __fadd_rn(A.B, 0.0f), PR = __fadd_rn(A.B, __fmul_rn((float)g.R, g.geom[12 * lev + 3 + a]));
        in = in & (moves | ((P0 <= ray.o[a]) & (ray.o[a] < PR)));
        m.A[a] = A;
    }
    return in & (m.E < m.X);
}

// Walk-order voxel owning t (inclusive = false) or the parameters just after
// t (inclusive = true) on a moving axis: the largest w with T(w) < t (resp.
// <=), first - 1 if none, first + R beyond the grid; from an estimate.
__device__ __forceinline__ bool crossed(float T, float t, bool inclusive) { return (T < t) | (inclusive & (T == t)); }
__device__ __forceinline__ int start_estimate(const WalkAxis &A, int first, int R, float t) {
    const float q = floorf((t - A.T(first)) * A.per);
    return first + (int)fminf(fmaxf(q, -1.0f), (float)R);   // a NaN becomes -1
}
__device__ __forceinline__ int start_exact(const WalkAxis &A, int w, int first, int R, float t, bool inclusive) {
    while (w >= first && !crossed(A.T(w), t, inclusive)) --w;
    while (w < first + R && crossed(A.T(w + 1), t, inclusive)) ++w;
    return w;
}
// On an axis that does not move: the voxel holding o, P(v) <= o < P(v+1); -1
// below the grid, R above it.
__device__ __forceinline__ int start_still(float B, float h, float inv_h, int R, float o) {
    const auto plane = [&](int v) { return __fadd_rn(B, __fmul_rn((float)v, h)); };
    int v = (int)fminf(fmaxf(floorf((o - B) * inv_h), -1.0f), (float)R);
    while (v >= 0 && plane(v) > o) --v;
    while (v < R && plane(v + 1) <= o) ++v;
    return v;
}

// Puts the cursor of level `lev` on the voxel owning t_min when t_min lies
// after the segment start a, else on the voxel owning the parameters just
// after a.  False when that voxel is outside the grid.
template <int kGrid, class Vis>
__device__ __forceinline__ bool cursor_begin(typename CursorOf<kGrid>::type &c, const GridView &g, const Tree &tree,
                                             int lev, const Ray &ray, const RayLevel &m, float a, const Lattice &lat,
                                             Vis &vis) {
    const int R = g.R;
    vis.begin_level(g, lev, ray.o, ray.d);
    const bool after = lat.tmin > a;
    const float ts = after ? lat.tmin : a;
    int w[3];
    bool sure = true;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const int first = m.A[q].flip & -R;
        w[q] = start_estimate(m.A[q], first, R, ts);
        const bool moves = axis_moves(ray.d[q], ray.r[q]);
        const bool enters = crossed(m.A[q].T(w[q]), ts, !after), leaves = crossed(m.A[q].T(w[q] + 1), ts, !after);
        sure = sure & moves & enters & !leaves;
    }
    if (!sure) {
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            if (axis_moves(ray.d[q], ray.r[q]))
                w[q] = start_exact(m.A[q], w[q], m.A[q].flip & -R, R, ts, !after);
            else
                w[q] = start_still(m.A[q].B, g.geom[12 * lev + 3 + q], g.geom[12 * lev + 6 + q], R, ray.o[q]);
        }
    }
    bool in = true;
#pragma unroll
    for (int q = 0; q < 3; ++q) in = in & ((uint32_t)(w[q] ^ m.A[q].flip) < (uint32_t)R);
    if (!in) return false;
    c.A0 = m.A[0];
    c.A1 = m.A[1];
    c.A2 = m.A[2];
    if constexpr (kGrid == 0) {
        c.start(g.bits, (uint64_t)lev * R * R * R, R, w[0], w[1], w[2]);
    } else if constexpr (kGrid == 2) {
        c.dist = g.dist + (uint64_t)lev * R * R * R;
        c.R = R;
        c.slack = relocate_slack(g.geom, lev, R, ray.o, lat.tmax);
        c.w0 = w[0];
        c.w1 = w[1];
        c.w2 = w[2];
        c.lookup();
    } else {
        c.t = tree;
        c.lev = lev;
        c.set_node(tree.root[tree.NR == 1 ? lev : 0]);   // of the level's only root cell, else set by the lookup
        c.slack = relocate_slack(g.geom, lev, R, ray.o, lat.tmax);
        c.w0 = w[0];
        c.w1 = w[1];
        c.w2 = w[2];
        c.Dm1 = 0;
        c.lblk = -1;
        c.code = 0;
        c.lu4 = 0;
        c.lookup(a);
    }
    return true;
}

// m: the level as the ray meets it (its axes are used, not its span)
template <int kGrid, bool kSkip, class Vis, class Ctx>
__device__ __forceinline__ void march_segment(const GridView &g, const Tree &tree, int lev, const Ray &ray,
                                              const RayLevel &m, float a, float b, const Lattice &lat, Vis &vis,
                                              const Ctx &ctx) {
    typename CursorOf<kGrid>::type c;
    if (!cursor_begin<kGrid>(c, g, tree, lev, ray, m, a, lat, vis)) return;
    drive<kSkip>(c, a, b, lat.tmax, vis, ctx);
}

// A single-level ray before its walk: hit is false for a ray with no samples
// to find (it misses the grid, the span lies outside [t_min, t_max],
// t_min > t_max, or the origin or direction is not finite).
struct L1Span {
    Ray ray;
    RayLevel m;
    bool hit;
};

__device__ __forceinline__ L1Span l1_span(const GridView &g, const float o[3], const float d[3], const Lattice &lat) {
    L1Span s{};
    bool ok = lat.tmin <= lat.tmax;
#pragma unroll
    for (int a = 0; a < 3; ++a) ok = ok && __builtin_isfinite(o[a]) && __builtin_isfinite(d[a]);
    s.ray = make_ray(o, d);
    s.hit = meet_level(g, 0, s.ray, s.m) & ok & (s.m.E < lat.tmax) & (s.m.X >= lat.tmin);
    return s;
}

// Issue priority of a wave from the dense-step estimate of its longest ray:
// sum over axes of |d_a| * len / h_a, with len its span's length inside
// [t_min, t_max], against the grid's resolution R (a ray through the grid
// crosses between R and 3R planes).  The waves of long rays walk longest --
// on a camera looking at an object, the image's centre tiles run for the
// whole launch while most waves end early -- so letting them issue first
// when several waves of a SIMD are ready shortens the launch, and the short
// waves fill the gaps.  The level is made wave-uniform (readfirstlane), so
// the wave takes one scalar branch.  All 64 lanes must call it together.
__device__ __forceinline__ void set_wave_priority(float nv, int R) {
    if (!(nv >= 0.0f)) nv = 0.0f;
#pragma unroll
    for (int k = 32; k >= 1; k >>= 1) nv = fmaxf(nv, __shfl_xor(nv, k));
    const float r = (float)R;
    const int lvl = __builtin_amdgcn_readfirstlane(nv > 1.65f * r ? 3 : nv > 1.15f * r ? 2 : nv > 0.6f * r ? 1 : 0);
    if (lvl == 3) __builtin_amdgcn_s_setprio(3);
    else if (lvl == 2) __builtin_amdgcn_s_setprio(2);
    else if (lvl == 1) __builtin_amdgcn_s_setprio(1);
}

// A ray may be walked in parts, each by a lane of its own, that meet at
// parameters between its first and last: part j of n holds (c_j, c_{j+1}]
// with c_0 = -inf and c_n = +inf, and walks as if the ray began after c_j.
// Parts of one ray compute a shared c from the same inputs with the same
// operations, so they agree on it to the bit, and every parameter belongs to
// exactly one part.
struct RayPart {
    int j, n;
};

// All samples of one part of a ray, in increasing t.  The cascade boxes are
// nested (checked when the grid is built), so level l holds exactly
// (E_l, X_l] and these intervals nest.  With f the finest level the ray meets
// and m = L-1-f, segment k = 0..2m runs in t order: for k < m level L-1-k on
// (E_{L-1-k}, E_{L-2-k}]; for k = m level f on (E_f, X_f]; for k > m level
// f+(k-m) on (X_{f+k-m-1}, X_{f+k-m}].  Each segment is marched by its level.
// kL1: the grid has a single level (no cascades), so the level geometry is
// uniform across the wave.
//
// The parts share a ray's range evenly by the voxels it crosses: over one
// level evenly in t, over cascades by length over voxel size.

// Clips the span (a, b] of a one-level ray to a part of it.
__device__ __forceinline__ void clip_to_part(RayPart part, const Lattice &lat, float &a, float &b) {
    const float t0 = fmaxf(a, lat.tmin), len = __fsub_rn(fminf(b, lat.tmax), t0), each = 1.0f / (float)part.n;
    const auto c = [&](int j) { return __fadd_rn(t0, __fmul_rn(len, __fmul_rn((float)j, each))); };
    if (part.j > 0) a = fmaxf(a, c(part.j));
    if (part.j + 1 < part.n) b = fminf(b, c(part.j + 1));
}

template <int kGrid, bool kSkip, class Vis, class Ctx>
__device__ __forceinline__ void march_l1(const GridView &g, const Tree &tree, const L1Span &s, RayPart part,
                                         const Lattice &lat, Vis &vis, const Ctx &ctx) {
    float a = s.m.E, b = s.m.X;
    if (part.n > 1) {
        clip_to_part(part, lat, a, b);
        if (!(a < b)) return;
    }
    march_segment<kGrid, kSkip>(g, tree, 0, s.ray, s.m, a, b, lat, vis, ctx);
}

template <int kGrid, bool kSkip, bool kL1 = false, class Vis, class Ctx>
__device__ __forceinline__ void trace_ray(const GridView &g, const Tree &tree, const float o[3], const float d[3],
                                          RayPart part, const Lattice &lat, Vis &vis, const Ctx &ctx) {
    if (kL1) {
        const L1Span s = l1_span(g, o, d, lat);
        if (s.hit) march_l1<kGrid, kSkip>(g, tree, s, part, lat, vis, ctx);
        return;
    }
    if (!(lat.tmin <= lat.tmax)) return;
#pragma unroll
    for (int a = 0; a < 3; ++a)
        if (!__builtin_isfinite(o[a]) || !__builtin_isfinite(d[a])) return;
    const Ray ray = make_ray(o, d);
    const int L = g.L;
    const auto clip = [&](float t) { return fminf(fmaxf(t, lat.tmin), lat.tmax); };
    // voxels of level lev per unit of t, up to a factor the levels share
    const auto density = [&](int lev) { return g.geom[12 * lev + 6]; };
    int f = -1;
    float work = 0.0f;    // the ray's range in voxels (parts only)
    float inner_len = 0.0f;
    for (int lev = 0; lev < L && (f < 0 || part.n > 1); ++lev) {
        RayLevel m;
        if (meet_level(g, lev, ray, m)) {
            if (f < 0) f = lev;
            const float len = clip(m.X) - clip(m.E);
            work += fmaxf(len - inner_len, 0.0f) * density(lev);
            inner_len = len;
        }
    }
    if (f < 0) return;
    const float each = work / (float)part.n;
    const float from = __fmul_rn((float)part.j, each), to = __fmul_rn((float)(part.j + 1), each);
    float done = 0.0f;    // voxels before the segment
    const int m = L - 1 - f;
    // Every lane first passes the segments it has nothing to do in, then
    // marches: the lanes of a wave (parts of a ray, or rays that enter
    // through different levels) march their own segments side by side.
    for (int k = 0; k <= 2 * m;) {
        RayLevel at;
        int lev = 0;
        float a = 0.0f, b = 0.0f;
        bool found = false;
        for (; k <= 2 * m && !found; ++k) {
            // the two levels whose spans bound segment k
            lev = k < m ? L - 1 - k : f + (k - m);
            RayLevel in;
            meet_level(g, k == m ? f : lev - 1, ray, in);
            meet_level(g, lev, ray, at);
            a = k <= m ? at.E : in.X;
            b = k < m ? in.E : at.X;
            if (part.n > 1 && L == 1) {
                // as the walk of one-level grids cuts it, to the bit: a part
                // counted there may be walked again here
                clip_to_part(part, lat, a, b);
            } else if (part.n > 1) {
                // Both parts beside a boundary w get the same cut of the segment
                // from it, and cuts rise with w: whatever the lengths and their
                // rounding are, each parameter falls to one part.  A segment
                // that adds nothing to `done` (no length inside [t_min, t_max],
                // as every one of a ray with near = far) goes whole to one part.
                const float t0 = clip(a), len = __fsub_rn(clip(b), t0), here = __fmul_rn(len, density(lev));
                const float before = done, next = __fadd_rn(done, here);
                const auto cut = [&](float w) {
                    if (w <= before) return a;
                    return w < next ? fminf(fmaxf(__fadd_rn(t0, __fmul_rn(len, (w - before) / here)), a), b) : b;
                };
                const float a_part = part.j > 0 ? cut(from) : a;
                b = part.j + 1 < part.n ? cut(to) : b;
                a = a_part;
                done = next;
            }
            found = a < b && b >= lat.tmin && a < lat.tmax;
        }
        if (found) march_segment<kGrid, kSkip>(g, tree, lev, ray, at, a, b, lat, vis, ctx);
    }
}

// ------------------------------------------------------------------ expansion fill

// Expansion fill: the output range [offsets[r0], offsets[r0 + 256]) of 256
// consecutive rays (a chunk) is cut into windows of 4-output groups, and a
// block writes its share of them with consecutive lanes on consecutive groups
// (full-wave 16-byte stores).  The rays' kept runs are staged
// in LDS in output order with block-relative first outputs; a ray whose runs
// were lost contributes one placeholder run over its outputs, which the
// traversal fill writes instead, so the runs tile the outputs without gaps.
// The owner of every group comes from a map built per window of groups:
// each run marks the group holding its first output with its index (LDS
// max), and a block-wide max-scan then names, for every group, the last run
// starting at or before its last output.  A lane reads its group's owner and
// looks back over at most three earlier runs; there is no per-output search.
// The run starting last before a window marks the window's first group, so
// each window's map stands alone.  Marks carry the window's number in their
// high bits, so the map is cleared once per chunk: entries left by earlier
// windows are smaller than the current window's first mark.
// The windows of a chunk (2048 groups each, counted from the chunk's first
// group) are dealt round-robin to kExpandParts blocks, so a chunk dense with
// samples does not run its windows one after another in one block while the
// rest of the chip has finished.
// Outputs counted from the chunk's first group fit in 32 bits: a ray has fewer
// than 2^24 samples, so 256 rays and the three outputs before them stay below
// 2^32.
// A group looks at most four runs back and reads each output's run whole (first
// index and ray, 8 bytes); a growing step's points come from LDS when they
// fit, so that the write loop issues no global load: one counter covers
// loads and stores on this architecture, and a load waits for every store
// before it.  A 1280 x 832 frame on four cascades with 244 million samples
// went from 709 to 561 us (5.2 TB/s of output), with the points in LDS.  Scans
// by the vector unit's lane moves and run slots loaded four at a time took 1 to
// 1.5 us off every block: a 64 x 64 frame's expansion 9.4 to 8.0 us.
// Tried beside it: the same work by single waves, 64 rows each, without any
// barrier (20 to 50% slower on frames, whose rows with many samples then sit
// in few waves, 5% slower with the samples dealt out evenly).
constexpr int kExpandRuns = 1024;     // runs staged per pass
constexpr int kExpandGroups = 2048;   // 4-output groups per owner window
constexpr int kExpandParts = 4;       // blocks sharing one chunk's windows
// Waves per SIMD asked of the expansion kernels: six blocks of 256 lanes per CU
// (LDS allows seven, without a table).  At the register budget this leaves (80 VGPRs) the
// expansion keeps its loops free of spills; only the rarely taken lost-ray
// traversal spills (the -O1 build; at -O2 the growing-step path spilled as
// well).  An expansion block
// spends much of its life waiting on loads and barriers while the other
// blocks' stores fill HBM, so residency is what keeps the writes flowing.
constexpr int kExpandWaves = 6;
constexpr int kTableLds = 4096;       // growing-step lattice points kept in LDS, at most
constexpr int kGroupsPerLane = kExpandGroups / kBlock;
constexpr int kOwnerBits = 11;        // owner entries: window number << 11 | (1 + run), run < 1024
// The owner map is padded with one word after every kGroupsPerLane entries:
// the max-scan has lane t read entries kGroupsPerLane*t .. +kGroupsPerLane-1,
// which then sit at words 9t .. 9t+7; with 9 odd, the 32 lanes an LDS access
// serves at a time meet 32 different banks (unpadded, stride 8 put four lanes
// on every bank).
constexpr int kOwnSlots = kExpandGroups + kExpandGroups / kGroupsPerLane;
__device__ __forceinline__ int own_slot(int g) { return g + g / kGroupsPerLane; }

struct OneLattice {       // every ray on one lattice
    static constexpr bool kMulti = false;
    Lattice lat;
};

struct SceneLattices {    // ray r on the lattice of its scene
    static constexpr bool kMulti = true;
    const Lattice *lats;   // [n]
    const int64_t *first;  // first global ray of each scene, [n + 1]
    int n;
    // of a wave-uniform ray
    __device__ __forceinline__ int scene_of(int64_t r) const {
        int s = 0;
        for (int b = 1; b < n; b += 64) {
            const int k = b + (int)(threadIdx.x & 63);
            s += __popcll(__ballot(k < n && first[min(k, n)] <= r));
        }
        return s;
    }
};

struct RunReader {
    const int2 *slots;    // [kMaxRuns][stride]
    int64_t stride;
    const int32_t *ray_next;
    const int2 *chunks;
    const int32_t *chunk_next;
};

// Inclusive scans over the 64 lanes: row shifts by 1, 2, 4, 8, then lane 15 of a
// row of 16 to the next of rows 1 and 3, and lane 31 to rows 2 and 3 (lanes that
// nothing is moved to add 0).  Through the vector unit's own lane moves these
// take a tenth of the time of six exchanges through LDS.
template <int kCtrl, int kRows>
__device__ __forceinline__ int32_t lanes_moved(int32_t v) {
    return __builtin_amdgcn_update_dpp(0, v, kCtrl, kRows, 0xf, false);
}
template <class Step>
__device__ __forceinline__ void wave_scan_steps(const Step &step) {
    using std::integral_constant;
    step(integral_constant<int, 0x111>{}, integral_constant<int, 0xf>{});
    step(integral_constant<int, 0x112>{}, integral_constant<int, 0xf>{});
    step(integral_constant<int, 0x114>{}, integral_constant<int, 0xf>{});
    step(integral_constant<int, 0x118>{}, integral_constant<int, 0xf>{});
    step(integral_constant<int, 0x142>{}, integral_constant<int, 0xa>{});
    step(integral_constant<int, 0x143>{}, integral_constant<int, 0xc>{});
}
__device__ __forceinline__ int64_t wave_scan(int64_t v) {
    wave_scan_steps([&](auto ctrl, auto rows) {
        const int32_t lo = lanes_moved<decltype(ctrl)::value, decltype(rows)::value>((int32_t)v);
        const int32_t hi = lanes_moved<decltype(ctrl)::value, decltype(rows)::value>((int32_t)(v >> 32));
        v += (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
    });
    return v;
}
__device__ __forceinline__ int32_t wave_scan(int32_t v) {
    wave_scan_steps([&](auto ctrl, auto rows) { v += lanes_moved<decltype(ctrl)::value, decltype(rows)::value>(v); });
    return v;
}
__device__ __forceinline__ uint32_t wave_scan_max(uint32_t v) {
    wave_scan_steps([&](auto ctrl, auto rows) {
        v = max(v, (uint32_t)lanes_moved<decltype(ctrl)::value, decltype(rows)::value>((int32_t)v));
    });
    return v;
}

// The scan done inside the expansion (one-call sampling, and rays walked in
// parts, whose rows the offsets array does not list): every block derives
// its 256-row chunk's offsets from the count pass's per-ray counts, counted
// from its sums per 4096-ray scan tile and per 256-ray chunk, and the first part
// of every chunk writes them to the offsets array (the last chunk also the total
// and the overflow flag); or, with the rays' offsets given (write == 0), counted
// from the given offset of the chunk's first ray, so that a fill writes where its
// offsets say.
constexpr int kChunksPerTile = kScanTile / kBlock;
struct ChunkScan {
    const int32_t *counts;       // [n_rays] (rows)
    const int64_t *tile_sums;    // [ceil(n_rays / kScanTile)]
    const int64_t *chunk_sums;   // [ceil(n_rays / kBlock)]
    int32_t *overflow;           // nullable: set to (total > capacity)
    int32_t parts_log2;          // log2 of a ray's rows: the rows of ray i are i << parts_log2 ...
    int32_t write;               // 0: the offsets array is given, and not written
};

// First output of row i (for the rare rows the count pass could not keep runs
// for; a plain sequential sum): from the sums, or, where the offsets are given,
// from its ray's and the counts of the ray's rows before it.
__device__ inline int64_t offset_of_row(int64_t i, const ChunkScan &cs, const int64_t *offsets) {
    int64_t s = 0, r = i / kBlock * kBlock;
    if (cs.write != 0) {
        const int64_t c = i / kBlock, T = i / kScanTile;
        for (int64_t k = 0; k < T; ++k) s += cs.tile_sums[k];
        for (int64_t j = T * kChunksPerTile; j < c; ++j) s += cs.chunk_sums[j];
    } else {
        r = i >> cs.parts_log2 << cs.parts_log2;
        s = offsets[i >> cs.parts_log2];
    }
    for (; r < i; ++r) s += cs.counts[r];
    return s;
}

// Inclusive block scan of x (returned, with its total) and the block sum of
// y, sharing one exchange through LDS (lds holds 2 * kBlock / 64 entries, not
// written again before a barrier).
__device__ __forceinline__ int64_t block_scan_and_sum256(int64_t x, int64_t y, int64_t *lds, int64_t &x_total,
                                                        int64_t &y_total) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    x = wave_scan(x);
    y = wave_scan(y);
    if (lane == 63) {
        lds[wid] = x;
        lds[kBlock / 64 + wid] = y;
    }
    __syncthreads();
    int64_t below = 0;
    x_total = 0;
    y_total = 0;
#pragma unroll
    for (int w = 0; w < kBlock / 64; ++w) {
        const int64_t v = lds[w];
        if (w < wid) below += v;
        x_total += v;
        y_total += lds[kBlock / 64 + w];
    }
    return below + x;
}
__device__ __forceinline__ int32_t block_scan256(int32_t x, int32_t *lds, int32_t &total) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    x = wave_scan(x);
    if (lane == 63) lds[wid] = x;
    __syncthreads();
    int32_t below = 0;
    total = 0;
#pragma unroll
    for (int w = 0; w < kBlock / 64; ++w) {
        const int32_t v = lds[w];
        if (w < wid) below += v;
        total += v;
    }
    return below + x;
}

// A staged run: its first lattice index less its first output (mod 2^32: output
// p has lattice index bn + p), and its ray (-1: a lost ray's placeholder).
struct RunBody {
    uint32_t bn;
    int32_t ray;
};

// LDS of one expansion block.
struct ExpandLds {
    uint32_t start[kExpandRuns + 1];   // first output; [cn] bounds the last run of the pass
    RunBody body[kExpandRuns];
    uint32_t own[kOwnSlots];           // 1 + owner run of each group of the window, at own_slot(group)
    uint32_t wmax[kBlock / 64];
    int32_t runs[kBlock / 64];
    int64_t wave[2 * (kBlock / 64)];
};

// Points of a lattice: computed (constant step, kTable false), or read from a
// table in LDS or in global memory.
template <bool kTable>
struct Points {
    float tmin, dt;
    const float *tab;
    int n_tab;
    __device__ __forceinline__ void at(int n, int32_t, float &a, float &b) const {
        if constexpr (kTable) {
            // outputs beside the written ones are looked up too
            n = min(max(n, 0), n_tab - 2);
            a = tab[n];
            b = tab[n + 1];
        } else {   // Lattice::t of a constant step
            const float f = (float)n;
            a = __fadd_rn(tmin, __fmul_rn(f, dt));
            b = __fadd_rn(tmin, __fmul_rn(f + 1.0f, dt));
        }
    }
};

// Points of a chunk of rows that several scenes share: each by its ray's scene.
struct ScenePoints {
    const Lattice *lats;
    const uint8_t *scene;   // [kBlock], in LDS: of each row
    int64_t r0;             // first row's ray
    __device__ __forceinline__ void at(int n, int32_t ray, float &a, float &b) const {
        a = b = 0.0f;
        if (ray < 0) return;   // a placeholder
        const Lattice L = lats[scene[ray - r0]];
        if (!L.cone) Points<false>{L.tmin, L.dt, nullptr, 0}.at(n, ray, a, b);
        // a growing step with far < near has no table, and its rays no samples
        else if (L.n_tab > 0) Points<true>{L.tmin, L.dt, L.tab, L.n_tab}.at(n, ray, a, b);
    }
};

// What a block knows of its chunk.  Outputs are counted from the chunk's first
// group of four (absolute output 4 * g0).
struct ChunkOut {
    int64_t g0;
    uint32_t lim;          // outputs end here (chunk's end or capacity)
    uint32_t end;          // the chunk's outputs end here
    uint32_t start, len;   // the lane's row's outputs
    int64_t row;
    int32_t ray;
    int nr;                // its runs to stage (kRunsLost: lost), 0 if the part needs none of it
    int2 s0, s1;           // the first two
};

// Writes the outputs of the part's windows.  Entered and left by the whole block.
template <class P>
__device__ __forceinline__ void expand_windows(ExpandLds &sh, const ChunkOut &ch, int part,
                                               const RunReader &rd, const P &pts, int32_t *__restrict__ ray_ids,
                                               float *__restrict__ t0, float *__restrict__ t1, bool vec4) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    int nr = ch.nr;
    int32_t ray = ch.ray;
    int2 s0 = ch.s0;
    if (nr == kRunsLost) {
        nr = ch.len > 0 ? 1 : 0;
        s0 = make_int2(0, (int)ch.len);
        ray = -1;
    }
    for (int i = threadIdx.x; i < kOwnSlots; i += kBlock) sh.own[i] = 0;
    int32_t total;
    const int rb = block_scan256(nr, sh.runs, total) - nr;
    uint32_t epoch = 0;   // window number within the block
    for (int c0 = 0; c0 < total; c0 += kExpandRuns) {
        const int cn = min(total - c0, kExpandRuns);
        // stage runs c0 .. c0+cn-1; slot cn takes the next pass's first start.
        uint32_t st = ch.start;
        auto stage = [&](int k, int2 rn) {
            const int idx = rb + k - c0;
            if (idx >= 0 && idx <= cn) {
                sh.start[idx] = st;
                if (idx < cn) sh.body[idx] = RunBody{(uint32_t)rn.x - st, ray};
            }
            st += (uint32_t)(rn.y - rn.x);
        };
        if (nr > 0) stage(0, s0);
        if (nr > 1) stage(1, ch.s1);
        if (nr > 2) {   // two, then four at a time, their loads together
            const int2 r2 = rd.slots[2 * rd.stride + ch.row], r3 = rd.slots[3 * rd.stride + ch.row];
            stage(2, r2);
            if (nr > 3) stage(3, r3);
        }
        int32_t chunk = -1;
        for (int k = 4; k < nr; k += 4) {
            const int2 *src = rd.slots + (int64_t)k * rd.stride + ch.row;
            int64_t next = rd.stride;
            if (k >= kMaxRuns) {
                if (k % kMaxRuns == 0) chunk = k == kMaxRuns ? rd.ray_next[ch.row] : rd.chunk_next[chunk];
                src = rd.chunks + (int64_t)chunk * kMaxRuns + k % kMaxRuns;
                next = 1;
            }
            const int2 r0 = src[0], r1 = src[next], r2 = src[2 * next], r3 = src[3 * next];
            stage(k, r0);
            if (k + 1 < nr) stage(k + 1, r1);
            if (k + 2 < nr) stage(k + 2, r2);
            if (k + 3 < nr) stage(k + 3, r3);
        }
        if (threadIdx.x == 0 && c0 + cn == total) sh.start[cn] = ch.end;
        __syncthreads();
        const uint32_t lo = sh.start[0];
        const uint32_t hi = min(sh.start[cn], ch.lim);
        if (hi > lo) {
            // groups covering [lo, hi)
            const uint32_t g_first = lo >> 2, g_last = (hi - 1) >> 2;
            // this part's windows that meet the pass: w = part, part + kExpandParts, ...
            uint32_t w = g_first / kExpandGroups;
            w += ((uint32_t)part - w) % kExpandParts;
            for (; w * kExpandGroups <= g_last; w += kExpandParts) {
                const uint32_t gw = max(g_first, w * kExpandGroups);
                const int nwin = (int)(min(g_last, (w + 1) * kExpandGroups - 1) - gw + 1);
                const uint32_t tag = ++epoch << kOwnerBits;
                for (int a = threadIdx.x; a < cn; a += kBlock) {
                    const uint32_t g = sh.start[a] >> 2;
                    if (g >= gw + nwin) continue;
                    // a run starting before the window marks group 0 if it is the last such run
                    // (run 0 starts at or before gw, so group 0 always holds a mark of this window)
                    if (g >= gw || a + 1 == cn || (sh.start[a + 1] >> 2) >= gw)
                        atomicMax(&sh.own[own_slot(g > gw ? (int)(g - gw) : 0)], tag | (uint32_t)(a + 1));
                }
                __syncthreads();
                // block-wide inclusive max-scan of own
                uint32_t v[kGroupsPerLane];
                uint32_t m = 0;
#pragma unroll
                for (int e = 0; e < kGroupsPerLane; ++e) {
                    m = max(m, sh.own[(kGroupsPerLane + 1) * threadIdx.x + e]);
                    v[e] = m;
                }
                const uint32_t incl = wave_scan_max(m);
                if (lane == 63) sh.wmax[wid] = incl;
                uint32_t pre = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)incl, 0x138, 0xf, 0xf, false);   // lane below
                __syncthreads();
                for (int q = 0; q < wid; ++q) pre = max(pre, sh.wmax[q]);
#pragma unroll
                for (int e = 0; e < kGroupsPerLane; ++e) sh.own[(kGroupsPerLane + 1) * threadIdx.x + e] = max(pre, v[e]);
                __syncthreads();
                // each lane writes groups k = tid, tid + 256, ... of the window
                const int64_t at = 4 * (ch.g0 + gw);
                int32_t *const wi = ray_ids + at;
                float *const w0 = t0 + at, *const w1 = t1 + at;
                for (int k = threadIdx.x; k < nwin; k += kBlock) {
                    const int a = (int)(sh.own[own_slot(k)] & ((1u << kOwnerBits) - 1)) - 1;   // owns the group's last output
                    const uint32_t p = 4 * (gw + (uint32_t)k);
                    // runs a-1, a-2, a-3 may own the group's earlier outputs
                    const uint32_t sa = sh.start[a], sb = sh.start[max(a - 1, 0)], sc = sh.start[max(a - 2, 0)];
                    int4 id;
                    float4 x0, x1;
                    auto one = [&](uint32_t j, int32_t &r, float &u, float &v) {
                        const RunBody b = sh.body[max(a - (int)(sa > j) - (int)(sb > j) - (int)(sc > j), 0)];
                        r = b.ray;
                        pts.at((int)(b.bn + j), r, u, v);
                    };
                    one(p, id.x, x0.x, x1.x);
                    one(p + 1, id.y, x0.y, x1.y);
                    one(p + 2, id.z, x0.z, x1.z);
                    id.w = sh.body[a].ray;
                    pts.at((int)(sh.body[a].bn + p + 3), id.w, x0.w, x1.w);
                    if (vec4 && p >= lo && p + 3 < hi && (id.x | id.y | id.z | id.w) >= 0) {
                        reinterpret_cast<int4 *>(wi)[k] = id;
                        reinterpret_cast<float4 *>(w0)[k] = x0;
                        reinterpret_cast<float4 *>(w1)[k] = x1;
                    } else {   // an end, a placeholder, or no 16-byte stores
                        const int q = 4 * k;
                        if (p >= lo && p < hi && id.x >= 0) wi[q] = id.x, w0[q] = x0.x, w1[q] = x1.x;
                        if (p + 1 >= lo && p + 1 < hi && id.y >= 0) wi[q + 1] = id.y, w0[q + 1] = x0.y, w1[q + 1] = x1.y;
                        if (p + 2 >= lo && p + 2 < hi && id.z >= 0) wi[q + 2] = id.z, w0[q + 2] = x0.z, w1[q + 2] = x1.z;
                        if (p + 3 >= lo && p + 3 < hi && id.w >= 0) wi[q + 3] = id.w, w0[q + 3] = x0.w, w1[q + 3] = x1.w;
                    }
                }
                __syncthreads();
            }
        }
        __syncthreads();
    }
    if (total == 0) __syncthreads();   // own and runs are free for the next use
}

template <bool kScan, class Lats>
__device__ __forceinline__ void expand_chunk(ExpandLds &sh, const float *table_lds, int64_t r0, int part,
                                             int64_t *__restrict__ offsets, const ChunkScan &cs, int64_t n_rays,
                                             const int32_t *__restrict__ nruns, const RunReader &rd,
                                             const Lats &lats, int64_t capacity, int32_t *__restrict__ ray_ids,
                                             float *__restrict__ t0, float *__restrict__ t1, bool vec4) {
    const int64_t r = r0 + threadIdx.x;
    const bool in = r < n_rays;
    const int64_t rc = in ? r : n_rays - 1;   // lanes past the last ray load a valid one's
    int64_t base, bend, off, off_next;
    if constexpr (kScan) {
        // every load here depends on r alone and is issued in one round: the
        // sums before the chunk (whole tiles, then the earlier chunks of its
        // tile) and the ray's count; the run count and run slots follow once
        // the scan shows whether the ray's outputs meet this part's windows
        const int64_t c = r0 / kBlock, T = r0 / kScanTile;
        if (part > 0) {
            // the chunk's outputs span at most (count + 6) / 4 groups, wherever
            // they start: a part beyond them has no window (and part 0, which
            // writes the chunk's offsets, always goes on)
            if ((cs.chunk_sums[c] + 6) / 4 <= (int64_t)part * kExpandGroups) return;
        }
        int64_t before = 0;
        if (cs.write != 0) {
            for (int64_t k = threadIdx.x; k < T; k += kBlock) before += cs.tile_sums[k];
            const int64_t j = T * kChunksPerTile + threadIdx.x;
            if (j < c) before += cs.chunk_sums[j];
        } else if (threadIdx.x == 0) {
            before = offsets[r0 >> cs.parts_log2];   // a chunk's rows are those of whole rays
        }
        const int64_t cnt = in ? (int64_t)cs.counts[r] : 0;
        int64_t total;
        const int64_t incl = block_scan_and_sum256(cnt, before, sh.wave, total, base);
        off = base + incl - cnt;
        off_next = base + incl;
        bend = base + total;
        if (part == 0 && cs.write != 0) {
            if (in && (r & ((1 << cs.parts_log2) - 1)) == 0) offsets[r >> cs.parts_log2] = off;
            if (r0 + kBlock >= n_rays && threadIdx.x == 0) {
                offsets[n_rays >> cs.parts_log2] = bend;
                if (cs.overflow) *cs.overflow = bend > capacity ? 1 : 0;
            }
        }
    } else {
        // the chunk's bounds first (uniform loads): a part with no window of
        // the chunk returns before it reads anything per ray
        base = offsets[r0];
        bend = offsets[min(r0 + kBlock, n_rays)];
    }
    const int64_t lim = min(bend, capacity);
    const int64_t G0 = base >> 2;   // the chunk's first group; windows count from it
    if (lim <= base || (((lim - 1) >> 2) - G0) / kExpandGroups < part) {   // block-uniform: nothing to write
        if constexpr (kScan) __syncthreads();   // sh.wave is free for the next item
        return;
    }
    ChunkOut ch;
    ch.g0 = G0;
    const int64_t origin = 4 * G0;
    ch.lim = (uint32_t)(lim - origin);
    ch.end = (uint32_t)(bend - origin);
    ch.row = r;
    ch.ray = (int32_t)(kScan ? r >> cs.parts_log2 : r);
    // Every other global load of the staging depends on r alone, so all of
    // them are issued here together: one memory round trip (the ray's offsets
    // and run count, and its first two run slots, read whether or not the ray
    // has them; the slot arrays have a column for every ray).
    if constexpr (!kScan) {
        off = offsets[rc];
        off_next = offsets[rc + 1];
        ch.nr = nruns[rc];
        ch.s0 = rd.slots[rc];
        ch.s1 = rd.slots[rd.stride + rc];
        if (!in) ch.nr = 0;
    } else {
        // With the offsets computed here, a part stages only the rays whose
        // outputs meet one of its windows (w = part, part + kExpandParts, ...),
        // and only those rays' run counts and first run slots are read: the
        // windows are tiled by such rays, and the other parts write the rest.
        // This cuts the expansion's reads by more than half.  The three-call
        // form, whose offsets come from memory, measured slower with it and
        // keeps every ray.
        bool needed = in && off_next > off;
        if (needed) {
            const int64_t wa = ((off >> 2) - G0) / kExpandGroups, wb = (((off_next - 1) >> 2) - G0) / kExpandGroups;
            needed = wa + ((part - (int)(wa % kExpandParts)) + kExpandParts) % kExpandParts <= wb;
        }
        ch.nr = 0;
        ch.s0 = ch.s1 = make_int2(0, 0);
        if (needed) {
            ch.nr = nruns[rc];
            ch.s0 = rd.slots[rc];
            ch.s1 = rd.slots[rd.stride + rc];
        }
    }
    ch.start = in ? (uint32_t)(off - origin) : 0u;
    ch.len = in ? (uint32_t)(off_next - off) : 0u;
    auto write = [&](const Lattice &L, bool in_lds) {
        if (!L.cone)
            expand_windows(sh, ch, part, rd, Points<false>{L.tmin, L.dt, nullptr, 0}, ray_ids, t0, t1, vec4);
        else if (in_lds)
            expand_windows(sh, ch, part, rd, Points<true>{L.tmin, L.dt, table_lds, L.n_tab}, ray_ids, t0, t1, vec4);
        else
            expand_windows(sh, ch, part, rd, Points<true>{L.tmin, L.dt, L.tab, L.n_tab}, ray_ids, t0, t1, vec4);
    };
    if constexpr (Lats::kMulti) {
        // nearly every chunk lies in one scene; scene by scene, a chunk of many
        // small ones would be written once for each (64 scenes of 4 rays: 482 us)
        __shared__ uint8_t scene[kBlock];
        int sc = lats.scene_of(r0);
        if (lats.first[sc + 1] >= min(r0 + kBlock, n_rays)) {
            write(lats.lats[sc], false);
        } else {
            while (lats.first[sc + 1] <= rc) ++sc;
            scene[threadIdx.x] = (uint8_t)sc;
            __syncthreads();
            expand_windows(sh, ch, part, rd, ScenePoints{lats.lats, scene, r0}, ray_ids, t0, t1, vec4);
        }
    } else {
        write(lats.lat, lats.lat.n_tab <= kTableLds);
    }
}

// Work items are (256-ray chunk, part) pairs, kExpandParts per chunk, part
// by part: item i is part i / chunks of chunk i % chunks.  Blocks go to the
// XCDs round-robin, so this order gives every XCD an even share of part 0
// (which every chunk with samples has) instead of sending all of it to the
// XCDs whose index is a multiple of kExpandParts.  The grid strides over the
// items, so a launch may use fewer blocks than items (every item ends on a
// barrier or returns before its first one, so its LDS is free for the next).
__host__ __device__ inline int64_t expand_items(int64_t n_rays) {
    return (n_rays + kBlock - 1) / kBlock * kExpandParts;
}

template <bool kScan = false, class Lats>
__device__ __forceinline__ void expand_block(int64_t *__restrict__ offsets, const ChunkScan &cs, int64_t n_rays,
                                             const int32_t *__restrict__ nruns, const RunReader &rd,
                                             const Lats &lats, int64_t capacity, int32_t *__restrict__ ray_ids,
                                             float *__restrict__ t0, float *__restrict__ t1, bool vec4, float *table_lds) {
    __shared__ ExpandLds sh;
    if constexpr (!Lats::kMulti) {
        const Lattice &L = lats.lat;
        if (L.cone && L.n_tab <= kTableLds) {
            for (int i = threadIdx.x; i < L.n_tab; i += kBlock) table_lds[i] = L.tab[i];
            __syncthreads();
        }
    }
    const int64_t chunks = (n_rays + kBlock - 1) / kBlock;
    for (int64_t it = blockIdx.x; it < chunks * kExpandParts; it += gridDim.x)
        expand_chunk<kScan>(sh, table_lds, it % chunks * kBlock, (int)(it / chunks), offsets, cs, n_rays, nruns, rd,
                            lats, capacity, ray_ids, t0, t1, vec4);
}

// ------------------------------------------------------------------ ray order

// The width a call's image is tiled by: a row longer than the call has rays is cut
// to them (only whole tiles of no ray are left out, of which an image width far
// beyond the rays would launch any number).
inline int tiled_width(int64_t n, int width) { return (int)std::min<int64_t>(width, std::max<int64_t>(n, 1)); }

// Threads per image-tiled launch: 8x8-pixel tiles of 64 lanes (one wave);
// with rays walked in parts, 2^parts_log2 threads a ray.
__host__ __device__ inline int64_t tiled_threads(int64_t n, int width, int parts_log2 = 0) {
    if (width <= 0) return ((n + 63) / 64 * 64) << parts_log2;
    const int64_t rows = (n + width - 1) / width;
    return (((width + 7) / 8) * ((rows + 7) / 8) * (int64_t)64) << parts_log2;
}

// Ray walked by thread t: t itself, or with an image of `width` pixels per
// row, lane l of wave w takes pixel (8*(w % tiles_x) + l % 8, 8*(w / tiles_x)
// + l / 8) of the row-major image; -1 for a lane past the image.
__device__ __forceinline__ int64_t ray_of_thread(int64_t t, int64_t n, int width) {
    if (width <= 0) return t < n ? t : -1;
    const int64_t w = t >> 6;
    const int l = (int)(t & 63);
    const int64_t tiles_x = (width + 7) >> 3;
    const int64_t px = (w % tiles_x) * 8 + (l & 7);
    const int64_t py = (w / tiles_x) * 8 + (l >> 3);
    if (px >= width) return -1;
    const int64_t r = py * width + px;
    return r < n ? r : -1;
}

// The same with rays walked in parts: the lowest lane_log2 bits of a ray's
// part number vary across neighbouring lanes, the others across waves.
__device__ __forceinline__ int64_t ray_of_thread(int64_t t, int64_t n, int width, int parts_log2, int lane_log2,
                                                 RayPart &part) {
    const int wave_log2 = parts_log2 - lane_log2;
    const int64_t w = t >> 6;
    const int l = (int)(t & 63);
    // the wave's slice of 64 >> lane_log2 rays of a tile (or of 64 consecutive rays)
    const int64_t slice = w >> wave_log2;
    part.n = 1 << parts_log2;
    part.j = (int)(w & ((1 << wave_log2) - 1)) << lane_log2 | (l & ((1 << lane_log2) - 1));
    return ray_of_thread(slice << (6 - lane_log2) | (l >> lane_log2), n, width);
}

// ------------------------------------------------------------------ ray loads

__device__ __forceinline__ void load_ray(const float *origins, const float *dirs, int64_t i, float o[3], float d[3]) {
    o[0] = origins[3 * i + 0];
    o[1] = origins[3 * i + 1];
    o[2] = origins[3 * i + 2];
    d[0] = dirs[3 * i + 0];
    d[1] = dirs[3 * i + 1];
    d[2] = dirs[3 * i + 2];
}

}  // namespace ogv
