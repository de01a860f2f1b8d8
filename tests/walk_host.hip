// The ray walk of trace.hpp compiled for the host, for tests that need no GPU:
// a dense grid's rays walked whole and in parts, and relocations.
// Only what the walk itself uses of the device's builtins is given a host form.
#include <hip/hip_runtime.h>

#include <type_traits>

#undef __device__
#define __device__ __attribute__((device)) __attribute__((host))
#undef __shared__
#define __shared__ static
#define __builtin_amdgcn_rcpf(x) (1.0f / (x))
static int products;   // of plane crossings computed so far
#define __fmul_rn(a, b) (++products, (a) * (b))
#define __fadd_rn(a, b) ((a) + (b))
#define __fsub_rn(a, b) ((a) - (b))
#define __fdiv_rn(a, b) ((a) / (b))

#include "../paper_2404_10272_amd/csrc/trace.hpp"

using namespace ogv;

namespace {

// Keeps the occupied runs (lo, hi] of a walk.
struct Runs {
    float *out;
    int n, cap;
    __device__ void begin_level(const GridView &, int, const float *, const float *) {}
    __device__ bool room(const Lattice &) { return true; }
    __device__ void make_room(const Lattice &) {}
    __device__ void run(const Lattice &, float lo, float hi) {
        if (n < cap) {
            out[2 * n] = lo;
            out[2 * n + 1] = hi;
        }
        ++n;
    }
};

}  // namespace

// Runs of part j of n of a ray on a dense grid, at most cap of them in out
// [cap][2]; returns their number.  single: by the walk of one-level grids.
extern "C" int walk_runs(int L, int R, const float *geom, const uint32_t *bits, const float *o, const float *d,
                         float near_t, float far_t, int j, int n, int single, float *out, int cap) {
    GridView g{};
    g.kind = 0;
    g.L = L;
    g.R = R;
    g.geom = geom;
    g.bits = bits;
    Lattice lat{};
    lat.tmin = near_t;
    lat.tmax = far_t;
    lat.dt = 1.0f;
    Runs runs{out, 0, cap};
    if (single) trace_ray<0, false, true>(g, Tree{}, o, d, RayPart{j, n}, lat, runs, lat);
    else trace_ray<0, false, false>(g, Tree{}, o, d, RayPart{j, n}, lat, runs, lat);
    return runs.n;
}

// Relocation of a ray of a one-level grid that steps at t out of a cell of voxels
// w[a] .. p[a]-1; returns the products it computed beside the estimates.
extern "C" int relocation(int R, const float *geom, const float *o, const float *d, int *w, const int *p, float t) {
    WalkAxis A[3];
    for (int a = 0; a < 3; ++a) A[a] = walk_axis(geom, 0, a, o[a], d[a], 1.0f / d[a]);
    const float T[3] = {A[0].T(p[0]), A[1].T(p[1]), A[2].T(p[2])};
    products = 0;
    relocate(A[0], A[1], A[2], w[0], w[1], w[2], p[0], p[1], p[2], T[0], T[1], T[2], t, relocate_slack(geom, 0, R, o, 100.0f));
    return products;
}
