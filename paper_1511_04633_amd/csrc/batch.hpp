// batch.hpp -- one launch advancing many cavities of different size and
// parameters by one time step (same node update as k_step: pull streaming
// with the wall rules of Eqs. 6-10, double-MRT collision of Sec. 3).
//
// Work list: every active cavity's nodes, in storage order and each plane filled up
// to whole wavefronts (slots), are cut into tiles of blockDim.x slots; tile t is
// {cavity, first slot}.  A block takes tiles blockIdx.x, blockIdx.x + gridDim.x, ...
// (grid-stride "persistent" blocks when gridDim.x is smaller than the tile count, one
// tile per block when equal).  A wavefront's nodes are consecutive in every
// population segment and start on a memory line, so its stores cover whole lines,
// and it is full except at the end of a plane.  (Tiles over the nodes alone put
// wavefronts across lines where n^2 is no multiple of 64: us per step, FP16, 6 of
// 50^3 20.5, 3 of 100^3 72.2; here 16.6 and 54.8.)  The per-cavity table (lattice pointers,
// geometry, relaxation rates) is read with wavefront-uniform loads.
#pragma once

#include "kernels.hpp"

namespace lbmx {

template <typename T>
struct BatchCav {
    char *lat[2];        // the cavity's two lattices
    Geometry<T> geo;
    Rates<T> rates;
    uint32_t plane;      // slots of a plane: n^2 up to a multiple of 64 (n of them < 2^24)
    float inv_n, inv_plane;  // their reciprocals, for the quotients below
};

// Slots of a plane of n^2 nodes.
__host__ __device__ constexpr uint32_t plane_slots(uint32_t n) { return (n * n + 63) / 64 * 64; }

struct Tile {
    uint32_t cav;        // index into the cavity table
    uint32_t start;      // first slot
};

// Each cavity's time step lives on the device, in two arrays used by turns:
// a launch of parity p reads cavity k's step from t_in[k] (the stochastic-
// rounding key of the fixed-point energy format, the same key a lone
// cavity uses at that step) and the block that owns the cavity's first
// tile writes step + 1 to t_out[k], which the next launch (parity 1 - p)
// reads.  No launch writes what it reads, so a captured graph replays with
// advancing steps.
template <class St, int kForce, int kPolicy>
__global__ __launch_bounds__(1024) void k_step_batch(const BatchCav<typename St::T> *__restrict__ cavs,
                                                     const Tile *__restrict__ tiles, uint32_t ntiles,
                                                     int parity, const uint32_t *__restrict__ t_in,
                                                     uint32_t *__restrict__ t_out)
{
    using T = typename St::T;
    for (uint32_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
        const Tile tile = tiles[t];
        const BatchCav<T> *cv = cavs + tile.cav;
        const uint32_t step = t_in[tile.cav];
        if (tile.start == 0 && threadIdx.x == 0)
            t_out[tile.cav] = step + 1u;
        const uint32_t n = uint32_t(cv->geo.n), slot = tile.start + threadIdx.x;
        const uint32_t z = div_small(slot, cv->plane, cv->inv_plane), cp = slot - z * cv->plane;
        if (cp >= n * n || z >= n)
            continue;
        const uint32_t q = div_small(cp, n, cv->inv_n);
        const int x = int(cp - q * n), y = int(q);
        const Geometry<T> geo = cv->geo;
        Site s = site_in_plane<St>(int(n), x, y, int(z));
        const uint32_t plane = z * Plane<St>(n).bytes;
        s.vF += plane;
        s.vG += plane;
        T f[19], g[7];
        pull<St, true>(cv->lat[parity], geo, s, y, f, g);
        collide<T, kForce>(f, g, cv->rates);
        put<St, kPolicy>(cv->lat[parity ^ 1], s, cp + n * n * z, step, geo, f, g);
    }
}

// Trilinear resampling of node-centred fields (n^3, x fastest) onto an
// m^3 node-centred grid covering the same cube; positions outside the
// outermost node centres are clamped to them.  out[k][m^3] for the fields
// in[k][n^3], k < nf.
__global__ __launch_bounds__(256) void k_resample(const double *__restrict__ in, int n, int nf,
                                                  float *__restrict__ out, int m)
{
    const long long c = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long mc = (long long)m * m * m;
    if (c >= mc)
        return;
    const int o[3] = {int(c % m), int((c / m) % m), int(c / ((long long)m * m))};
    int i0[3], i1[3];
    double fr[3];
    for (int d = 0; d < 3; ++d) {
        double p = (o[d] + 0.5) * double(n) / double(m) - 0.5;
        p = fmin(fmax(p, 0.0), double(n - 1));
        int k = int(floor(p));
        if (k > n - 2) k = n - 2 < 0 ? 0 : n - 2;
        i0[d] = k;
        i1[d] = k + 1 < n ? k + 1 : n - 1;
        fr[d] = p - k;
    }
    const size_t cells = (size_t)n * n * n;
    for (int k = 0; k < nf; ++k) {
        const double *a = in + (size_t)k * cells;
        auto at = [&](int x, int y, int z) { return a[x + (size_t)n * (y + (size_t)n * z)]; };
        const double c00 = at(i0[0], i0[1], i0[2]) * (1 - fr[0]) + at(i1[0], i0[1], i0[2]) * fr[0];
        const double c10 = at(i0[0], i1[1], i0[2]) * (1 - fr[0]) + at(i1[0], i1[1], i0[2]) * fr[0];
        const double c01 = at(i0[0], i0[1], i1[2]) * (1 - fr[0]) + at(i1[0], i0[1], i1[2]) * fr[0];
        const double c11 = at(i0[0], i1[1], i1[2]) * (1 - fr[0]) + at(i1[0], i1[1], i1[2]) * fr[0];
        const double c0 = c00 * (1 - fr[1]) + c10 * fr[1];
        const double c1 = c01 * (1 - fr[1]) + c11 * fr[1];
        out[(size_t)k * mc + c] = float(c0 * (1 - fr[2]) + c1 * fr[2]);
    }
}

}  // namespace lbmx
