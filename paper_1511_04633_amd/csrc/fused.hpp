// fused.hpp -- two time steps of one cavity in one pass over memory.
//
// k_step is bound by HBM from about 100^3 on (26 populations in and out per
// node and step, at the rate its access pattern reaches) and by its launch
// below about 40^3.  The kernels here take a block of nodes through two steps
// between one read and one write of the lattice: step A (time t) on the block
// and a one-node halo, its post-collision populations into LDS, step B (time
// t + 1) from LDS.  Halo nodes are updated by every block that needs them; each
// node update is the same inlined code as k_step and the values in LDS are the
// values k_step would have stored, so the result is k_step's bit for bit (the
// storage must hold populations in the arithmetic type: FP32 and FP64).
#pragma once

#include <algorithm>

#include "kernels.hpp"

namespace lbmx {

// Keep a node's values in registers at this point: nothing that computes them
// moves past it, so that the compiler contracts multiplications and additions
// as in k_step, where the whole update is one block of straight-line code.
template <typename T>
__device__ __forceinline__ void pin(T (&f)[19], T (&g)[7])
{
#pragma unroll
    for (int i = 0; i < 19; ++i)
        asm volatile("" : "+v"(f[i]));
#pragma unroll
    for (int i = 0; i < 7; ++i)
        asm volatile("" : "+v"(g[i]));
}

// The work item of a block: workgroup i runs on XCD i mod 8, and each XCD takes
// a contiguous eighth of the items, so that neighbouring tiles, whose halos
// overlap, are read through one L2.
__device__ __forceinline__ int xcd_item()
{
    const int b = int(blockIdx.x), nb = int(gridDim.x), xcd = b % 8;
    return xcd * (nb / 8) + min(xcd, nb % 8) + b / 8;
}

// ------------------------------------------------------------- small grids
// One tile of tx x ty x tz nodes per block; step A runs on the tile and its
// halo (clipped at the walls) with one thread per node, at most NT of them.
// Bound by launch and memory latency: 16^3 FP32 3.65 us per step with k_step,
// 2.65 us here; 32^3 4.25 -> 3.2 us.
template <class St, int kForce, int NT>
__global__ __launch_bounds__(NT) void
k_step2_tile(const char *__restrict__ src, char *__restrict__ dst, Geometry<typename St::T> geo,
             Rates<typename St::T> rates, int tx, int ty, int tz, int ntx, int nty)
{
    using T = typename St::T;
    __shared__ T lf[19 * NT], lg[7 * NT];
    const int n = geo.n, tid = threadIdx.x;
    const int item = xcd_item();
    const int bz = item / (ntx * nty), bt = item - bz * (ntx * nty), by = bt / ntx, bx = bt - by * ntx;
    const int x0 = bx * tx, y0 = by * ty, z0 = bz * tz;
    const int xl = max(x0 - 1, 0), yl = max(y0 - 1, 0), zl = max(z0 - 1, 0);
    const int hw = min(x0 + tx + 1, n) - xl, hh = min(y0 + ty + 1, n) - yl, hd = min(z0 + tz + 1, n) - zl;
    const uint32_t plane = Plane<St>(uint32_t(n)).bytes;
    {
        const int r = tid / hw, hx = tid - r * hw, hz = r / hh, hy = r - hz * hh;
        if (hz < hd) {
            const int x = xl + hx, y = yl + hy, z = zl + hz;
            Site s = site_in_plane<St>(n, x, y, z);
            s.vF += uint32_t(hz) * plane;
            s.vG += uint32_t(hz) * plane;
            T f[19], g[7];
            pull<St, true>(src + size_t(plane) * zl, geo, s, y, f, g);
            collide<T, kForce>(f, g, rates);
            pin(f, g);
#pragma unroll
            for (int i = 0; i < 19; ++i)
                lf[i * NT + tid] = f[i];
#pragma unroll
            for (int i = 0; i < 7; ++i)
                lg[i * NT + tid] = g[i];
        }
    }
    __syncthreads();
    const int bw = min(x0 + tx, n) - x0, bh = min(y0 + ty, n) - y0, bd = min(z0 + tz, n) - z0;
    const int r = tid / bw, cx = tid - r * bw, cz = r / bh, cy = r - cz * bh;
    if (cz >= bd)
        return;
    const int x = x0 + cx, y = y0 + cy, z = z0 + cz;
    Site s = site_in_plane<St>(n, x, y, z);
    const int q0 = (x - xl) + hw * ((y - yl) + hh * (z - zl));
    auto at = [&](int i) {  // the slot of population i's source, as in load_pops
        const int ex = ex19(i), ey = ey19(i), ez = ez19(i);
        const bool out = (ex > 0 && s.xl) || (ex < 0 && s.xh) || (ey > 0 && s.yl) || (ey < 0 && s.yh) ||
                         (ez > 0 && s.zl) || (ez < 0 && s.zh);
        return out ? opp19(i) * NT + q0 : i * NT + q0 - ex - hw * (ey + hh * ez);
    };
    RawPops<St> raw;
#pragma unroll
    for (int i = 0; i < 19; ++i)
        raw.f[i] = lf[at(i)];
#pragma unroll
    for (int i = 0; i < 7; ++i)
        raw.g[i] = lg[at(i)];
    T f[19], g[7];
    decode_pops<St, true, true>(raw, geo, s, y, f, g);
    collide<T, kForce>(f, g, rates);
    s.vF += uint32_t(cz) * plane;
    s.vG += uint32_t(cz) * plane;
    put<St, kNear>(dst + size_t(plane) * z0, s,
                   uint32_t(x) + uint32_t(n) * (uint32_t(y) + uint32_t(n) * uint32_t(z)), geo.step + 1u, geo, f, g);
}

// ------------------------------------------------------------- large grids
// A block marches through planes z0 - 1 .. z1 of a column of TX x TY nodes: in
// one turn it runs step A on plane z (TX + 2 by TY + 2 nodes, one thread each)
// and step B on plane z - 1 (TX by TY).  LDS holds what step B still needs:
// the populations with e_z = -1 of plane z, those with e_z = 0 of plane z - 1
// and those with e_z = +1 of planes z - 2 and z - 1 (by the parity of z): 32
// values per node of the halo rectangle instead of 3 x 26, so that 990 FP32
// nodes fit one CU's 160 KB.  A turn: step A in registers, its e_z = -1 values
// to LDS, barrier, step B gathers, barrier, the other values to LDS over those
// just read, step B collides and stores.  The next plane's populations are
// loaded before step B's collision and waited for after it and before its
// stores, so that their latency overlaps the arithmetic and no load waits
// behind a store.
//
// Walls: step A writes a population that step B would pull from outside (the
// reflected opposite one, with the wall temperature applied) into the slot in
// which step B looks for it; step B has no wall conditions.
//
// Bound by HBM and by the memory phases that the barriers keep apart from the
// arithmetic (vector unit busy about half of the time; 256^3 FP32 reads 1.89 GB
// for 1.74 GB of lattice).  256^3: FP32 581 -> 382 us per step, FP64 1179 ->
// 773 us; 128^3 FP32 74 -> 63 us.  64 x 13 tiles rather than 32 x 28 or
// 32 x 13: the rows' end columns cost a memory line each (FP32 256^3 with an
// earlier alignment: 405, 477 and 430 us); loading the next plane before step A
// instead spills vector registers.  As it is, the uniform values of the loop's two
// copies (with and without walls) spill: 52 scalar registers in FP32, 107 in FP64.
__device__ __forceinline__ constexpr int slot19(int i)
{
    constexpr int v[19] = {5, 6, 7, 8, 9, 14, 0, 10, 11, 12, 13, 15, 16, 1, 2, 17, 18, 3, 4};
    return v[i];  // + 5 for e_z = +1 and odd planes
}
__device__ __forceinline__ constexpr int slot7(int i)
{
    constexpr int v[7] = {1, 2, 3, 4, 5, 6, 0};
    return v[i];  // + 1 for e_z = +1 and odd planes
}

template <class St, int TX, int TY>
struct MarchTile {
    static constexpr int HW = TX + 2, HH = TY + 2, NH = HW * HH;
    static constexpr int NS = NH + 1;                  // slot NH takes the idle lanes' writes
    static constexpr int kWaves = (NH + 63) / 64;      // step A
    static constexpr int kWavesB = (TX * TY + 63) / 64;
    typename St::T f[24 * NS], g[8 * NS];
};

template <class St, int kForce, int TX, int TY, bool kEdge>
__device__ __forceinline__ void march2(const char *__restrict__ src, char *__restrict__ dst,
                                       const Geometry<typename St::T> &geo,
                                       const Rates<typename St::T> &rates, int x0, int y0, int z0, int z1,
                                       MarchTile<St, TX, TY> &lds)
{
    using T = typename St::T;
    using Tile = MarchTile<St, TX, TY>;
    constexpr int HW = Tile::HW, HH = Tile::HH, NH = Tile::NH, NS = Tile::NS;
    const int n = geo.n, tid = threadIdx.x;
    const size_t plane = Plane<St>(uint32_t(n)).bytes;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // step A: node (x, y) of the halo rectangle; lanes outside the cavity
    // repeat the nearest node and write to slot NH
    const int hx = tid % HW, hy = tid / HW;
    const int x = x0 - 1 + hx, y = y0 - 1 + hy;
    const bool inA = tid < NH && x >= 0 && x < n && y >= 0 && y < n;
    const int xc = min(max(x, 0), n - 1), yc = min(max(y, 0), n - 1);
    const int pw = inA ? tid : NH;
    // step B: node (x0 + bx, y0 + by)
    const int bx = tid % TX, by = tid / TX;
    const bool inB = tid < TX * TY && x0 + bx < n && y0 + by < n;
    const int pb = inB ? (by + 1) * HW + bx + 1 : HW + 1;
    const Site sB = site_in_plane<St>(n, x0 + bx, y0 + by, 1);

    Site s = site_in_plane<St>(n, xc, yc, 1);
    RawPops<St> raw;
    auto load = [&](int z) {
        s.zl = z == 0, s.zh = z == n - 1;
        load_pops<St, false, kEdge>(src + plane * z, n, s, raw);
    };
    const int za = max(z0 - 1, 0), zlast = min(z1, n - 1);
    load(za);
    pin(raw.f, raw.g);
    for (int z = za; z <= z1; ++z) {
        T f[19], g[7];
        s.zl = z == 0, s.zh = z == n - 1;
        decode_pops<St, false, kEdge>(raw, geo, s, yc, f, g);
        collide<T, kForce>(f, g, rates);
        pin(f, g);
        if (z < n) {
#pragma unroll
            for (int i = 0; i < 19; ++i)
                if (ez19(i) < 0)
                    lds.f[slot19(i) * NS + pw] = f[i];
            lds.g[slot7(6) * NS + pw] = g[6];
        }
        const int par = z & 1;
        __syncthreads();
        T f2[19], g2[7];
        if (wave < Tile::kWavesB) {
#pragma unroll
            for (int i = 0; i < 19; ++i)
                f2[i] = lds.f[slot19(i) * NS + (ez19(i) > 0 ? 5 * NS * par : 0) + pb - ex19(i) - HW * ey19(i)];
#pragma unroll
            for (int i = 0; i < 7; ++i)
                g2[i] = lds.g[slot7(i) * NS + (ez19(i) > 0 ? NS * par : 0) + pb - ex19(i) - HW * ey19(i)];
        }
        __syncthreads();
        if (z < n) {
#pragma unroll
            for (int i = 0; i < 19; ++i)
                if (ez19(i) >= 0)
                    lds.f[slot19(i) * NS + (ez19(i) > 0 ? 5 * NS * par : 0) + pw] = f[i];
#pragma unroll
            for (int i = 0; i < 6; ++i)
                lds.g[slot7(i) * NS + (ez19(i) > 0 ? NS * par : 0) + pw] = g[i];
            if (kEdge || z == 0 || z == n - 1) {
                const int pm = par ^ 1;  // parity of plane z - 1
                const T th_lin = theta_linear(geo, yc);
                const bool xd = x_wall_dirichlet(geo.wall_type), zd = z_wall_dirichlet(geo.wall_type);
                const T two_w = T(0.25);
#pragma unroll
                for (int i = 1; i < 19; ++i) {
                    const int ex = ex19(i), ey = ey19(i), ez = ez19(i);
                    const bool out = (ex > 0 && x == 0) || (ex < 0 && x == n - 1) || (ey > 0 && y == 0) ||
                                     (ey < 0 && y == n - 1) || (ez > 0 && z == 0) || (ez < 0 && z == n - 1);
                    const bool in_tile = !((ex > 0 && hx == 0) || (ex < 0 && hx == HW - 1) ||
                                           (ey > 0 && hy == 0) || (ey < 0 && hy == HH - 1));
                    if (!(inA && out && in_tile))
                        continue;
                    const int q = tid - ex - HW * ey;
                    lds.f[slot19(i) * NS + (ez > 0 ? 5 * NS * pm : 0) + q] = f[opp19(i)];
                    if (i < 7) {
                        const T v = g[opp19(i)];
                        T r;
                        if (ey != 0)  // hot wall y = 0, cold wall y = H (Eqs. 6, 7)
                            r = two_w * (ey > 0 ? geo.theta_hot : geo.theta_cold) - v;
                        else
                            r = (ex != 0 ? xd : zd) ? two_w * th_lin - v : v;
                        lds.g[slot7(i) * NS + (ez > 0 ? NS * pm : 0) + q] = r;
                    }
                }
            }
        }
        load(min(z + 1, zlast));
        if (wave < Tile::kWavesB) {
            collide<T, kForce>(f2, g2, rates);
            pin(f2, g2);
        }
        pin(raw.f, raw.g);  // the loads have landed: the stores below are waited for by nothing
        if (z > z0 && inB)
            put<St, kFar>(dst + plane * (z - 1), sB,
                          uint32_t(x0 + bx) + uint32_t(n) * (uint32_t(y0 + by) + uint32_t(n) * uint32_t(z - 1)),
                          geo.step + 1u, geo, f2, g2);
    }
}

// Waves per SIMD that the registers must allow: 4 in FP32 (128 registers, 16
// waves per CU: one 64 x 13 block or two 32 x 13), 2 in FP64.
template <class St>
constexpr int march_waves() { return sizeof(typename St::T) == 8 ? 2 : 4; }

// Blocks: ntx x nty columns by chunks of zc planes (two more are read).
template <class St, int kForce, int TX, int TY>
__global__ __launch_bounds__(64 * (MarchTile<St, TX, TY>::kWaves))
    __attribute__((amdgpu_waves_per_eu(march_waves<St>()))) void
k_step2_march(const char *__restrict__ src, char *__restrict__ dst, Geometry<typename St::T> geo,
              Rates<typename St::T> rates, int ntx, int nty, int zc)
{
    __shared__ MarchTile<St, TX, TY> lds;
    const int item = xcd_item();
    const int bt = item % (ntx * nty), ck = item / (ntx * nty);
    const int x0 = (bt % ntx) * TX, y0 = (bt / ntx) * TY, z0 = ck * zc, z1 = min(z0 + zc, geo.n);
    // kEdge: a wall node lies in the tile or its halo
    if (x0 == 0 || x0 + TX >= geo.n - 1 || y0 == 0 || y0 + TY >= geo.n - 1)
        march2<St, kForce, TX, TY, true>(src, dst, geo, rates, x0, y0, z0, z1, lds);
    else
        march2<St, kForce, TX, TY, false>(src, dst, geo, rates, x0, y0, z0, z1, lds);
}

// ------------------------------------------------------------------- rule
// How two steps of an n^3 cavity are taken (kSingle: by k_step twice).
struct Step2Plan {
    enum Kind { kSingle, kTile, kWide, kNarrow } kind;
    int tx, ty, tz, ntx, nty;  // tz: planes per tile or chunk
    unsigned blocks;
};

// Tiles while a launch costs more than the halo's arithmetic (measured us per
// step, k_step -> tiles: FP32 16^3 3.65 -> 2.6, 32^3 4.2 -> 3.1, 40^3 5.1 ->
// 4.7, 44^3 5.7 -> 5.8; FP64 16^3 4.5 -> 3.3, 32^3 5.0 -> 4.1, 36^3 5.8 ->
// 7.2).  Above, the shape and chunk length that take the fewest turns, a partly
// filled round of blocks counting as a full one: a turn of the 64 x 13 tile
// took 8.6 to 9.9 us over 96^3 .. 320^3, of two 32 x 13 blocks on one CU 9.6 to
// 10.5 us (FP64, one block: 9.0 to 11.2 us); where rows do not start on 64-byte
// boundaries 10.0 to 11.6, 10.8 to 17.8 and 10.9 to 14.3 us.  k_step, at the rate
// it reaches from memory or, `near`, from the memory-side cache, where that is
// shorter (FP32: 96^3 28.8 us against 32.7, 112^3 50.1 against 49.4; 144^3 106
// against 100, 192^3 242 against 182; FP64: 88^3 50 against 44).
template <typename T>
inline Step2Plan plan_step2(int n, int cus, bool near)
{
    constexpr bool f64 = sizeof(T) == 8;
    auto up = [](int a, int b) { return (a + b - 1) / b; };
    auto make = [&](Step2Plan::Kind k, int tx, int ty, int tz) {
        const int ntx = up(n, tx), nty = up(n, ty);
        return Step2Plan{k, tx, ty, tz, ntx, nty, unsigned(ntx * nty * up(n, tz))};
    };
    if (n <= 32)
        return make(Step2Plan::kTile, n, 2, 2);
    if (!f64 && n <= 40)
        return make(Step2Plan::kTile, up(n, 2), 3, 2);
    const double rate = f64 ? (near ? 7.0e6 : 5.65e6) : (near ? 6.6e6 : 5.95e6);  // bytes per us
    const double single = 2.0 + 52.0 * sizeof(T) * double(n) * n * n / rate;
    Step2Plan best = make(Step2Plan::kSingle, 1, 1, 1);
    double best_us = 0.98 * single;
    const bool aligned = n % (f64 ? 8 : 16) == 0;
    for (int k = f64 ? 1 : 0; k < 2; ++k) {
        const int tx = k == 0 ? 64 : 32, ty = 13, slots = (k == 1 && !f64 ? 2 : 1) * cus;
        const double turn = f64 ? (aligned ? 10.2 : 13.3) : k == 0 ? (aligned ? 9.2 : 10.7) : (aligned ? 10.2 : 15.0);
        const int tiles = up(n, tx) * up(n, ty);
        for (int nz = 1; nz <= n / 4; ++nz) {
            const int zc = up(n, nz);
            const double us = 0.5 * turn * up(tiles * up(n, zc), slots) * (zc + 2);
            if (us < best_us) {
                best_us = us;
                best = make(k == 0 ? Step2Plan::kWide : Step2Plan::kNarrow, tx, ty, zc);
            }
        }
    }
    return best;
}

}  // namespace lbmx
