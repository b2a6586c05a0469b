// fused.hpp -- two time steps of one cavity in one pass over memory.
#pragma once

#include "kernels.hpp"

namespace lbmx {

// Slots of the plane buffers in LDS: populations with e_z = -1 (one plane),
// e_z = 0 (one plane), e_z = +1 (two planes, by the parity of z).
__device__ __forceinline__ constexpr int slot19(int i, int par)
{
    constexpr int v[19] = {5, 6, 7, 8, 9, 14, 0, 10, 11, 12, 13, 15, 16, 1, 2, 17, 18, 3, 4};
    return ez19(i) > 0 ? v[i] + 5 * par : v[i];
}
__device__ __forceinline__ constexpr int slot7(int i, int par)
{
    constexpr int v[7] = {1, 2, 3, 4, 5, 6, 0};
    return i == 5 ? v[i] + par : v[i];
}

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

template <class St, int kForce, int NT, int WEU>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(WEU))) void
k_step2_tile(const char *__restrict__ src, char *__restrict__ dst, Geometry<typename St::T> geo,
             Rates<typename St::T> rates, int tx, int ty, int tz, int ntx, int nty)
{
    using T = typename St::T;
    using SF = typename St::F;
    using SG = typename St::G;
    __shared__ typename Codec<SF>::Raw lf[19 * NT];
    __shared__ typename Codec<SG>::Raw lg[7 * NT];
    const int n = geo.n, tid = threadIdx.x;
    int bid = blockIdx.x;
    const int nb = gridDim.x;
    if (nb % 8 == 0)
        bid = (bid % 8) * (nb / 8) + bid / 8;
    const int bz = bid / (ntx * nty), bt = bid - bz * (ntx * nty), by = bt / ntx, bx = bt - by * ntx;
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
                lf[i * NT + tid] = Codec<SF>::enc(f[i], T(inv_w19(i)));
            if constexpr (std::is_same<SG, Fix16>::value) {
                const RoundBits rb(uint32_t(x) + uint32_t(n) * (uint32_t(y) + uint32_t(n) * uint32_t(z)), geo.step);
#pragma unroll
                for (int i = 0; i < 7; ++i)
                    lg[i * NT + tid] = Codec<SG>::enc_r(g[i], T(inv_w7(i)) * geo.inv_escale, rb.u16(i));
            } else {
#pragma unroll
                for (int i = 0; i < 7; ++i)
                    lg[i * NT + tid] = Codec<SG>::enc(g[i], T(inv_w7(i)));
            }
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
    RawPops<St> raw;
    auto at = [&](int i) {
        const int ex = ex19(i), ey = ey19(i), ez = ez19(i);
        const bool out = (ex > 0 && s.xl) || (ex < 0 && s.xh) || (ey > 0 && s.yl) || (ey < 0 && s.yh) ||
                         (ez > 0 && s.zl) || (ez < 0 && s.zh);
        return out ? opp19(i) * NT + q0 : i * NT + q0 - ex - hw * (ey + hh * ez);
    };
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
    put<St>(dst + size_t(plane) * z0, s,
            uint32_t(x) + uint32_t(n) * (uint32_t(y) + uint32_t(n) * uint32_t(z)), geo.step + 1u, geo, f, g);
}

template <class St, int kForce, int TX, int TY, int NW, int WEU, bool PF>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(WEU))) void
k_step2(const char *__restrict__ src, char *__restrict__ dst, Geometry<typename St::T> geo,
        Rates<typename St::T> rates, int ntx, int nty, int zc)
{
    using T = typename St::T;
    using SF = typename St::F;
    using SG = typename St::G;
    using RF = typename Codec<SF>::Raw;
    static_assert(std::is_same<typename Codec<SG>::Raw, T>::value, "energy held in T");
    constexpr int HW = TX + 2, HH = TY + 2, NH = HW * HH, NS = NH + 1;  // slot NH takes the idle lanes' writes
    constexpr int WB = (TX * TY + 63) / 64;
    static_assert(NW * 64 >= NH, "");
    __shared__ RF lf[24 * NS];
    __shared__ T lg[8 * NS];
    const int n = geo.n;
    int bid = blockIdx.x;
    const int nb = gridDim.x;
    if (nb % 8 == 0)
        bid = (bid % 8) * (nb / 8) + bid / 8;
    const int bt = bid % (ntx * nty), ck = bid / (ntx * nty);
    const int x0 = (bt % ntx) * TX, y0 = (bt / ntx) * TY;
    const int z0 = ck * zc, z1 = min(z0 + zc, n);
    const int za = max(z0 - 1, 0);
    const size_t plane = Plane<St>(uint32_t(n)).bytes;
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);

    const int tid = threadIdx.x;
    const int hx = tid % HW, hy = tid / HW;
    const int x = x0 - 1 + hx, y = y0 - 1 + hy;
    const bool inA = tid < NH && x >= 0 && x < n && y >= 0 && y < n;
    const int xc = min(max(x, 0), n - 1), yc = min(max(y, 0), n - 1);
    const int pw = inA ? tid : NH;
    const bool wall_xy = x0 == 0 || x0 + TX >= n || y0 == 0 || y0 + TY >= n;  // uniform
    const int bx = tid % TX, by = tid / TX;
    const bool inB = tid < TX * TY && x0 + bx < n && y0 + by < n;
    const int pb = inB ? (by + 1) * HW + bx + 1 : HW + 1;
    const Site sB = site_in_plane<St>(n, x0 + bx, y0 + by, 1);

    auto march = [&](auto edge) {
        constexpr bool kEdge = decltype(edge)::value;
        Site s = site_in_plane<St>(n, xc, yc, 1);
        RawPops<St> raw;
        auto load = [&](int z) {
            s.zl = z == 0, s.zh = z == n - 1;
            load_pops<St, false, kEdge>(src + plane * z, n, s, raw);
        };
        auto touch = [&]() {
#pragma unroll
            for (int i = 0; i < 19; ++i)
                asm volatile("" : "+v"(raw.f[i]));
#pragma unroll
            for (int i = 0; i < 7; ++i)
                asm volatile("" : "+v"(raw.g[i]));
        };
        if (PF)
            load(za);
        if (PF)
            touch();
        for (int z = za; z <= z1; ++z) {
            T f[19], g[7];
            if (!PF)
                load(min(z, n - 1));
            s.zl = z == 0, s.zh = z == n - 1;
            decode_pops<St, false, kEdge>(raw, geo, s, yc, f, g);
            collide<T, kForce>(f, g, rates);
            pin(f, g);
            if (z < n) {
#pragma unroll
                for (int i = 0; i < 19; ++i)
                    if (ez19(i) < 0)
                        lf[slot19(i, 0) * NS + pw] = Codec<SF>::enc(f[i], T(inv_w19(i)));
                lg[slot7(6, 0) * NS + pw] = g[6];
            }
            const int par = z & 1;
            __syncthreads();
            T f2[19], g2[7];
            if (wave < WB) {
#pragma unroll
            for (int i = 0; i < 19; ++i) {
                const int q = pb - ex19(i) - HW * ey19(i);
                f2[i] = Codec<SF>::dec(lf[slot19(i, 0) * NS + (ez19(i) > 0 ? 5 * NS * par : 0) + q], T(w19(i)));
            }
#pragma unroll
            for (int i = 0; i < 7; ++i) {
                const int q = pb - ex19(i) - HW * ey19(i);
                g2[i] = lg[slot7(i, 0) * NS + (i == 5 ? NS * par : 0) + q];
            }
            }
            __syncthreads();
            if (z < n) {
#pragma unroll
                for (int i = 0; i < 19; ++i)
                    if (ez19(i) >= 0)
                        lf[slot19(i, 0) * NS + (ez19(i) > 0 ? 5 * NS * par : 0) + pw] =
                            Codec<SF>::enc(f[i], T(inv_w19(i)));
#pragma unroll
                for (int i = 0; i < 6; ++i)
                    lg[slot7(i, 0) * NS + (i == 5 ? NS * par : 0) + pw] = g[i];
                if ((kEdge || z == 0 || z == n - 1)) {
                    // reflected populations, written where step B will look for them
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
                        if (inA && out && in_tile)
                            lf[slot19(i, 0) * NS + (ez > 0 ? 5 * NS * pm : 0) + tid - ex - HW * ey] =
                                Codec<SF>::enc(f[opp19(i)], T(inv_w19(opp19(i))));
                    }
#pragma unroll
                    for (int i = 1; i < 7; ++i) {
                        const int ex = ex19(i), ey = ey19(i), ez = ez19(i);
                        const bool out = (ex > 0 && x == 0) || (ex < 0 && x == n - 1) || (ey > 0 && y == 0) ||
                                         (ey < 0 && y == n - 1) || (ez > 0 && z == 0) || (ez < 0 && z == n - 1);
                        const bool in_tile = !((ex > 0 && hx == 0) || (ex < 0 && hx == HW - 1) ||
                                               (ey > 0 && hy == 0) || (ey < 0 && hy == HH - 1));
                        if (inA && out && in_tile) {
                            const T v = g[opp19(i)];
                            T r;
                            if (ey != 0)
                                r = two_w * (ey > 0 ? geo.theta_hot : geo.theta_cold) - v;
                            else
                                r = (ex != 0 ? xd : zd) ? two_w * th_lin - v : v;
                            lg[slot7(i, 0) * NS + (i == 5 ? NS * pm : 0) + tid - ex - HW * ey] = r;
                        }
                    }
                }
            }
            if (PF)
                load(min(z + 1, n - 1));
            if (wave < WB) {
                collide<T, kForce>(f2, g2, rates);
                pin(f2, g2);
            }
            if (PF)
                touch();
            if (z > z0 && inB)
                put<St>(dst + plane * (z - 1), sB,
                        uint32_t(x0 + bx) + uint32_t(n) * (uint32_t(y0 + by) + uint32_t(n) * uint32_t(z - 1)),
                        geo.step + 1u, geo, f2, g2);
        }
    };
    if (wall_xy)
        march(std::true_type{});
    else
        march(std::false_type{});
}

}  // namespace lbmx
