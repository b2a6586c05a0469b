// kernels.hpp -- HIP kernels of the double-MRT cavity step for gfx950.
//
// Data layout in HBM: two lattices (ping-pong).  Nodes are numbered
// c = x + n*(y + n*z), x fastest.  A lattice is a sequence of n planes (one
// per z); a plane holds 19 D3Q19 segments of n^2 flow elements followed by 7
// D3Q7 segments of n^2 energy elements (segment i holds population i of the
// plane's nodes, x fastest).  A wavefront therefore reads and writes 64
// consecutive elements per population, the 26 streams of a block lie within
// three planes (a few MB) instead of 26 regions n^3 elements apart, and the
// address of "population i of the node e_i upstream" is a uniform base (which
// plane, which segment, which shift) plus a per-lane offset that is the same
// for every population: the addresses cost no vector instruction per access.
//
// What a lattice holds: the post-collision populations f*(t-1), g*(t-1).
// The step kernel gathers ("pulls") them from the upstream neighbours, which
// is streaming (Eq. 14, Eq. 29) together with the wall conditions, then
// collides in registers and writes f*(t), g*(t) at the node itself (aligned
// stores).  Reads of the state at time t (fields, Nu, populations) perform
// the same pull without colliding.  Initialising a state S_0 therefore means
// writing the unique post-collision set whose pull gives S_0 ("unstream").
//
// Wall conditions in pull form (walls half way between nodes, at rest):
//   D3Q19: f_i(x) = f*_ibar(x) when x - e_i is outside (bounce-back, Eq. 8);
//   D3Q7 : g_i(x) = -g*_ibar(x) + 2 w_T,i theta_W on a Dirichlet wall,
//          g_i(x) =  g*_ibar(x) on an adiabatic wall.
// Each D3Q7 link crosses a single wall, so edges and corners need no rule.
#pragma once

#include <hip/hip_bf16.h>
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "collide.hpp"

namespace lbmx {

// ------------------------------------------------------------------ storage
// Codec<S>: how one population is held in HBM.  Flow populations are stored
// as offsets df = f - w_i, energy populations as g; the 16-bit formats store
// df / w_i and g / w_T,i (the population relative to its weight), which keeps
// every direction's stored value O(u) or O(theta).  `Raw` is the bit
// container: loads return it and dec() reinterprets its bits; `inv_w` is the
// exact reciprocal of the weight (3, 18, 36; 4, 8), so encoding multiplies
// instead of dividing.
template <typename S>
struct Codec;

template <>
struct Codec<double> {
    using Raw = double;
    template <typename T> static __device__ __forceinline__ T dec(Raw v, T) { return T(v); }
    template <typename T> static __device__ __forceinline__ Raw enc(T v, T) { return double(v); }
};

template <>
struct Codec<float> {
    using Raw = float;
    template <typename T> static __device__ __forceinline__ T dec(Raw v, T) { return T(v); }
    template <typename T> static __device__ __forceinline__ Raw enc(T v, T) { return float(v); }
};

template <>
struct Codec<__half> {
    using Raw = unsigned short;
    template <typename T> static __device__ __forceinline__ T dec(Raw v, T w)
    {
        return T(__half2float(__ushort_as_half(v))) * w;
    }
    template <typename T> static __device__ __forceinline__ Raw enc(T v, T inv_w)
    {
        return __half_as_ushort(__float2half_rn(float(v * inv_w)));
    }
};

template <>
struct Codec<__hip_bfloat16> {
    using Raw = unsigned short;
    template <typename T> static __device__ __forceinline__ T dec(Raw v, T w)
    {
        return T(__bfloat162float(__ushort_as_bfloat16(v))) * w;
    }
    template <typename T> static __device__ __forceinline__ Raw enc(T v, T inv_w)
    {
        return __bfloat16_as_ushort(__float2bfloat16(float(v * inv_w)));
    }
};

// Checkpoint files hold a lattice in slabs of 2^L consecutive nodes (19 flow
// segments of 2^L elements, then 7 energy segments); L by the flow element's
// bytes: 8 KB flow segments (2^10 FP64, 2^11 FP32, 2^12 16-bit elements).
__host__ __device__ constexpr int slab_shift_for(size_t flow_bytes)
{
    return flow_bytes >= 8 ? 10 : (flow_bytes == 4 ? 11 : 12);
}

// Fixed-point energy storage: g_i / (w_T,i Theta) as a signed 16-bit integer
// in units of 2^-15 (range +-1).  Theta is the power of two at or above
// 2 max(|theta_hot|, |theta_cold|) (1 for the walls at +-1/2), so that
// |g_i / w_T,i| = |theta (1 + 4 e_i.u)| + non-equilibrium part stays below
// Theta; the spacing is then 3.1e-5 Theta, uniform (FP16's is 1.2e-4 to 2.4e-4
// over the |g/w_T| = 0.25 .. 1 where the temperature signal lives).
// The step kernels round stochastically (enc_r): up with probability equal to
// the fraction below, so that a change smaller than one spacing per step is
// kept on average instead of being rounded away every step (the slow thermal
// drift would otherwise stall: with rounding to nearest a 2^-14 code's Nu
// error at 64^3, Ra 1e6 was 4.3e-3, with stochastic rounding 1.5e-5; 8
// random bits instead of 16 left a 3.6e-4 bias at steady state).
// Initialisation rounds to nearest (enc).  The weight arguments carry Theta
// (w_T,i Theta to decode, 1/(w_T,i Theta) to encode; exact, Theta being a
// power of two).  Finite values saturate at +-32767; -32768 encodes NaN, so
// that a diverging run still reports non-finite values.
struct Fix16 {
    short bits;
};

template <>
struct Codec<Fix16> {
    using Raw = unsigned short;
    template <typename T> static __device__ __forceinline__ T dec(Raw v, T w)
    {
        const short q = short(v);
        return q == -32768 ? T(NAN) : T(q) * (w * T(1.0 / 32768.0));
    }
    static __device__ __forceinline__ Raw pack(float q)
    {
        return Raw(short(fminf(fmaxf(q, -32767.0f), 32767.0f)));
    }
    template <typename T> static __device__ __forceinline__ Raw enc(T v, T inv_w)
    {
        const float x = float(v * inv_w) * 32768.0f;
        return x == x ? pack(rintf(x)) : Raw(0x8000);
    }
    // u16: 16 uniformly random bits, u = u16 / 2^16 in [0, 1).  Rounds up when
    // u < x - floor(x), i.e. with probability frac(x) (to 2^-16).  Every
    // operation here is exact (scaling by powers of two, floor, the
    // difference of nearby floats), so the result does not depend on how the
    // compiler contracts the arithmetic around it; floor(x + u) would round
    // the sum to the spacing of x (2^-9 at |x| = 2^14) and bias the rounding.
    template <typename T> static __device__ __forceinline__ Raw enc_r(T v, T inv_w, uint32_t u16)
    {
        const float x = float(v * inv_w) * 32768.0f;
        if (!(x == x))
            return Raw(0x8000);
        const float fl = floorf(x);
        const float u = float(u16) * (1.0f / 65536.0f);
        return pack(u < x - fl ? fl + 1.0f : fl);
    }
};

// Random bits for the stochastic rounding of node c's energy populations at
// step t: the MurmurHash3 finaliser (multiply-xorshift) of a combination of
// the two counters gives the first 32-bit word, xorshift32 (Marsaglia) the
// next three; each word serves two populations, 16 bits each.
// Deterministic: a run repeats exactly.
struct RoundBits {
    uint32_t w[4];
    __device__ __forceinline__ RoundBits(uint32_t c, uint32_t t)
    {
        uint32_t h = c * 0x9E3779B1u + t * 0xC2B2AE3Du;
        h ^= h >> 16;
        h *= 0x85EBCA6Bu;
        h ^= h >> 13;
        h *= 0xC2B2AE35u;
        h ^= h >> 16;
        h |= 1u;  // xorshift needs a nonzero state
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            w[k] = h;
            h ^= h << 13;
            h ^= h >> 17;
            h ^= h << 5;
        }
    }
    __device__ __forceinline__ uint32_t u16(int i) const
    {
        return (i & 1) ? (w[i >> 1] >> 16) : (w[i >> 1] & 0xffffu);
    }
};

// Element types of the flow (SF) and energy (SG) segments; T is the
// arithmetic type of the collision (FP64 only when both are FP64).
template <typename SF, typename SG>
struct Store {
    using F = SF;
    using G = SG;
    // the energy codec's weights carry the temperature scale Theta
    static constexpr bool kScaledG = std::is_same<SG, Fix16>::value;
    static constexpr int kSlabShift = slab_shift_for(sizeof(SF));
    using T = typename std::conditional<std::is_same<SF, double>::value &&
                                            std::is_same<SG, double>::value,
                                        double, float>::type;
};

// ---------------------------------------------------------- lattice tables
// D3Q19 (Eq. 12) and D3Q7 (Eq. 28) in the paper's order, 0-based.
__device__ __forceinline__ constexpr int ex19(int i)
{
    constexpr int v[19] = {0, 1, -1, 0, 0, 0, 0, 1, -1, 1, -1, 1, -1, 1, -1, 0, 0, 0, 0};
    return v[i];
}
__device__ __forceinline__ constexpr int ey19(int i)
{
    constexpr int v[19] = {0, 0, 0, 1, -1, 0, 0, 1, 1, -1, -1, 0, 0, 0, 0, 1, -1, 1, -1};
    return v[i];
}
__device__ __forceinline__ constexpr int ez19(int i)
{
    constexpr int v[19] = {0, 0, 0, 0, 0, 1, -1, 0, 0, 0, 0, 1, 1, -1, -1, 1, 1, -1, -1};
    return v[i];
}
__device__ __forceinline__ constexpr int opp19(int i)
{
    constexpr int v[19] = {0, 2, 1, 4, 3, 6, 5, 10, 9, 8, 7, 14, 13, 12, 11, 18, 17, 16, 15};
    return v[i];
}
// Eq. (18) and Eq. (31), with exact reciprocals.
__device__ __forceinline__ constexpr double w19(int i)
{
    return i == 0 ? 1.0 / 3.0 : (i < 7 ? 1.0 / 18.0 : 1.0 / 36.0);
}
__device__ __forceinline__ constexpr double w7(int i) { return i == 0 ? 0.25 : 0.125; }
__device__ __forceinline__ constexpr double inv_w19(int i) { return i == 0 ? 3.0 : (i < 7 ? 18.0 : 36.0); }
__device__ __forceinline__ constexpr double inv_w7(int i) { return i == 0 ? 4.0 : 8.0; }

// ---------------------------------------------------------------- arguments
template <typename T>
struct Geometry {
    int n;
    int wall_type;     // 1, 2, 3
    T theta_hot, theta_cold;
    uint32_t step;     // time step being written (stochastic-rounding stream)
    T escale;          // Theta of the fixed-point energy code (1 otherwise)
    T inv_escale;      // 1 / Theta (exact: Theta is a power of two)
};

// theta on a linear wall (Eqs. 9-10) at node height y: the crossing point of
// an x or z link has the node's y = j + 1/2.
template <typename T>
__device__ __forceinline__ T theta_linear(const Geometry<T> &geo, int y)
{
    return geo.theta_hot + (geo.theta_cold - geo.theta_hot) * (T(y) + T(0.5)) / T(geo.n);
}

// Dirichlet flags of the x and z walls for the three cavity types.
__device__ __forceinline__ bool x_wall_dirichlet(int wall_type) { return wall_type != 1; }
__device__ __forceinline__ bool z_wall_dirichlet(int wall_type) { return wall_type == 2; }

// ----------------------------------------------------------------- access
// Populations are read and written with buffer instructions: a uniform base
// (the resource), a uniform 32-bit offset (which population of which plane,
// shifted by which neighbour) and a per-lane 32-bit offset that is the same
// for every population, so an access costs no vector arithmetic.  The
// resource spans 4 GiB from its base; every address formed lies inside the
// lattice.
using Buffer = __amdgpu_buffer_rsrc_t;
__device__ __forceinline__ Buffer make_buffer(const char *base)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(base), short(0), int(0xffffffffu), 0x00020000);
}
// Cache policies of the stores (step_policy chooses).  kNear writes through the XCD's
// L2 (sc1), so that a kernel's end finds little to write back, and keeps the line in
// the 256 MB memory-side cache, where the next step reads it if one lattice and most
// of the other fit.  kStream marks the line as not needed again (nt); kFar is the
// same with sc1 for 8- and 2-byte populations, which measured 1 to 8 % faster where
// stores cover whole lines (4-byte ones did not).  us per step, kStream -> kNear:
// FP32 64^3 11.8 -> 9.5, 96^3 33.3 -> 28.8, 104^3 41.4 -> 37.4; FP64 50^3 11.6 ->
// 9.15, 80^3 39 -> 32; f16 / i16 64^3 7.3 -> 6.9, 96^3 20.3 -> 18.3, 128^3 40 -> 36.
// Plain stores, written back at the kernel's end: FP32 64^3 9.5, 48^3 6.9 (kNear
// 6.6), f16 / i16 64^3 8.1.
constexpr int kNear = 16, kFar = 18, kStream = 2;
template <typename S, int kPolicy>
constexpr int store_bits() { return kPolicy == kFar && sizeof(typename Codec<S>::Raw) == 4 ? kStream : kPolicy; }

// Loads return the storage bits (Codec<S>::Raw); Codec<S>::dec converts.
// They are temporal, as a wavefront's x-shifted reads share cache lines with its
// neighbours', except where step_policy asks for nt ones.
template <typename S, bool kNt = false>
__device__ __forceinline__ typename Codec<S>::Raw ld(Buffer b, uint32_t lane, uint32_t uniform)
{
    using R = typename Codec<S>::Raw;
    if constexpr (sizeof(R) == 8) {
        typedef uint32_t u2 __attribute__((ext_vector_type(2)));
        return __builtin_bit_cast(R, u2(__builtin_amdgcn_raw_buffer_load_b64(b, lane, uniform, kNt ? 2 : 0)));
    } else if constexpr (sizeof(R) == 4)
        return __builtin_bit_cast(R, __builtin_amdgcn_raw_buffer_load_b32(b, lane, uniform, kNt ? 2 : 0));
    else
        return __builtin_bit_cast(R, __builtin_amdgcn_raw_buffer_load_b16(b, lane, uniform, kNt ? 2 : 0));
}
template <typename S, int kPolicy>
__device__ __forceinline__ void st(Buffer b, uint32_t lane, uint32_t uniform, typename Codec<S>::Raw v)
{
    using R = typename Codec<S>::Raw;
    if constexpr (sizeof(R) == 8) {
        typedef uint32_t u2 __attribute__((ext_vector_type(2)));
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, v), b, lane, uniform, store_bits<S, kPolicy>());
    } else if constexpr (sizeof(R) == 4)
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), b, lane, uniform, store_bits<S, kPolicy>());
    else
        __builtin_amdgcn_raw_buffer_store_b16(v, b, lane, uniform, store_bits<S, kPolicy>());
}

// Bytes of a segment of n^2 elements: whole 128-byte lines, so that a
// wavefront's 64 consecutive nodes start on a line in every segment and its
// stores cover whole lines (FP32 steps at 75^3: 20.3 us unpadded, 18.2 us;
// 16-bit at 100^3: 24.9, 21.3 us), and one line more where a segment of 64 KB
// or above is a multiple of 4 KB: the 26 streams then do not start on the same
// memory channel (256^3: FP32 589 -> 583 us, FP16 + FP32 384 -> 365 us; small
// segments gain nothing, at 64^3 FP64 the line costs 5 %).
__host__ __device__ __forceinline__ constexpr uint32_t segment_bytes(uint32_t bytes)
{
    const uint32_t lines = (bytes + 127) / 128 * 128;
    return lines >= 65536 && lines % 4096 == 0 ? lines + 128 : lines;
}

// A plane: flow segment i at i * segF, energy segment i at offG + i * segG,
// the next plane at `bytes`.
template <class St>
struct Plane {
    static constexpr uint32_t bF = uint32_t(sizeof(typename St::F)), bG = uint32_t(sizeof(typename St::G));
    uint32_t segF, segG, offG, bytes;
    __host__ __device__ __forceinline__ explicit Plane(uint32_t n)
        : segF(segment_bytes(n * n * bF)), segG(segment_bytes(n * n * bG)), offG(19 * segF),
          bytes(offG + 7 * segG)
    {
    }
};

// Where a thread's node lies: the lane's byte offsets in a flow and in an energy
// segment 0 from an address that is uniform over the block, and the walls it is
// at.  The address is the node's plane (z uniform) or the lattice (z per lane,
// whose offsets then include z planes; the lattice is below 4 GiB).
struct Site {
    uint32_t vF, vG;
    bool xl, xh, yl, yh, zl, zh;  // on the walls x = 0, x = H, ...
};

template <class St>
__device__ __forceinline__ Site site_in_plane(int n, int x, int y, int z)
{
    Site s;
    s.vF = uint32_t(x + n * y) * Plane<St>::bF;
    s.vG = uint32_t(x + n * y) * Plane<St>::bG;
    s.xl = x == 0, s.xh = x == n - 1;
    s.yl = y == 0, s.yh = y == n - 1;
    s.zl = z == 0, s.zh = z == n - 1;
    return s;
}

// The energy populations that came from a wall: v, the reflected value, turns
// into 2 w_T theta_W - v at a Dirichlet wall and stays at an adiabatic one.
// kXY, kZ: whether a lane may be at an x or y wall, at a z wall.
template <typename T, bool kXY, bool kZ>
__device__ __forceinline__ void wall_energy(const Geometry<T> &geo, const Site &s, int y, T g[7])
{
    const T two_w = T(0.25);  // 2 w_T,i for the moving directions
    if (kXY) {
        if (s.yl)  // +y from the hot wall y = 0 (Eq. 6)
            g[3] = two_w * geo.theta_hot - g[3];
        if (s.yh)  // -y from the cold wall y = H (Eq. 7)
            g[4] = two_w * geo.theta_cold - g[4];
    }
    const bool xd = kXY && x_wall_dirichlet(geo.wall_type), zd = kZ && z_wall_dirichlet(geo.wall_type);
    if ((xd && (s.xl || s.xh)) || (zd && (s.zl || s.zh))) {
        const T th_lin = theta_linear(geo, y);
        if (xd && s.xl)
            g[1] = two_w * th_lin - g[1];
        if (xd && s.xh)
            g[2] = two_w * th_lin - g[2];
        if (zd && s.zl)
            g[5] = two_w * th_lin - g[5];
        if (zd && s.zh)
            g[6] = two_w * th_lin - g[6];
    }
}

// ------------------------------------------------------------------- pull
// Gather the populations of the node at `s` (height y) at time t from the
// post-collision lattice (time t-1): streaming plus wall conditions.
//
// Population i comes from the node x - e_i, or, where that is outside, from
// population ibar of the node itself (reflected at the wall).  Inside, the
// address is base + d_i + lane offset with a uniform d_i; a lane at a wall
// takes the offset that undoes d_i and selects segment ibar.  kLaneZ: z varies
// over the lanes (base is the lattice) instead of being uniform (base is the
// plane).  kEdge = false: no lane is at an x or y wall (kLaneZ: at any wall).  kNt:
// the loads' policy.
template <class St>
struct RawPops {
    typename Codec<typename St::F>::Raw f[19];
    typename Codec<typename St::G>::Raw g[7];
};

template <class St, bool kLaneZ, bool kEdge, bool kNt = false>
__device__ __forceinline__ void load_pops(const char *__restrict__ base, int n, const Site &s, RawPops<St> &r)
{
    Plane<St> pl{uint32_t(n)};
    uint32_t row = uint32_t(n);
    // keep the uniform offsets out of the registers between uses: they are
    // recomputed by the scalar unit (a caller's loop would hoist all of them)
    asm volatile("" : "+s"(pl.segF), "+s"(pl.segG), "+s"(pl.offG), "+s"(pl.bytes), "+s"(row));
    // Both offsets carry a bias of two planes, taken off the base, so that
    // neither is negative: the uniform one lies up to a plane and a row below
    // the node's plane, and a wall lane's undoes up to two planes.
    const uint32_t P = pl.bytes, bias = 2 * P;
    const Buffer buf = make_buffer(base - 4 * size_t(P));
    const uint32_t vF = s.vF + bias, vG = s.vG + bias;

    auto source = [&](int ex, int ey, int ez, uint32_t seg, uint32_t seg_opp, uint32_t el, uint32_t v,
                      uint32_t &d) -> uint32_t {
        d = bias + seg - ez * P - (ex + ey * row) * el;
        if (!kLaneZ && ((ez > 0 && s.zl) || (ez < 0 && s.zh)))
            d = bias + seg_opp;
        if (!kEdge || (ex == 0 && ey == 0 && (!kLaneZ || ez == 0)))
            return v;
        const bool out = (ex > 0 && s.xl) || (ex < 0 && s.xh) || (ey > 0 && s.yl) || (ey < 0 && s.yh) ||
                         (kLaneZ && ((ez > 0 && s.zl) || (ez < 0 && s.zh)));
        return out ? v + (bias + seg_opp - d) : v;
    };
#pragma unroll
    for (int i = 0; i < 19; ++i) {
        uint32_t d;
        const uint32_t v = source(ex19(i), ey19(i), ez19(i), i * pl.segF, opp19(i) * pl.segF, pl.bF, vF, d);
        r.f[i] = ld<typename St::F, kNt>(buf, v, d);
    }
#pragma unroll
    for (int i = 0; i < 7; ++i) {  // D3Q7 directions are the first 7 of D3Q19
        uint32_t d;
        const uint32_t v = source(ex19(i), ey19(i), ez19(i), pl.offG + i * pl.segG,
                                  pl.offG + opp19(i) * pl.segG, pl.bG, vG, d);
        r.g[i] = ld<typename St::G, kNt>(buf, v, d);
    }
}

template <class St, bool kLaneZ, bool kEdge>
__device__ __forceinline__ void decode_pops(const RawPops<St> &r, const Geometry<typename St::T> &geo,
                                            const Site &s, int y, typename St::T f[19], typename St::T g[7])
{
    using T = typename St::T;
#pragma unroll
    for (int i = 0; i < 19; ++i)
        f[i] = Codec<typename St::F>::dec(r.f[i], T(w19(i)));
    const T es = St::kScaledG ? geo.escale : T(1);
#pragma unroll
    for (int i = 0; i < 7; ++i)
        g[i] = Codec<typename St::G>::dec(r.g[i], T(w7(i)) * es);
    wall_energy<T, kEdge, kEdge || !kLaneZ>(geo, s, y, g);
}

template <class St, bool kLaneZ, bool kEdge = true, bool kNt = false>
__device__ __forceinline__ void pull(const char *__restrict__ base, const Geometry<typename St::T> &geo,
                                     const Site &s, int y, typename St::T f[19], typename St::T g[7])
{
    RawPops<St> r;
    load_pops<St, kLaneZ, kEdge, kNt>(base, geo.n, s, r);
    decode_pops<St, kLaneZ, kEdge>(r, geo, s, y, f, g);
}

// Write the 26 populations of node number `node` at `s` (post-collision values
// of step `step`).
template <class St, int kPolicy>
__device__ __forceinline__ void put(char *__restrict__ base, const Site &s, uint32_t node, uint32_t step,
                                    const Geometry<typename St::T> &geo, const typename St::T f[19],
                                    const typename St::T g[7])
{
    using T = typename St::T;
    using SF = typename St::F;
    using SG = typename St::G;
    Plane<St> pl{uint32_t(geo.n)};
    asm volatile("" : "+s"(pl.segF), "+s"(pl.segG), "+s"(pl.offG));  // as in load_pops
    const Buffer buf = make_buffer(base);
#pragma unroll
    for (int i = 0; i < 19; ++i)
        st<SF, kPolicy>(buf, s.vF, i * pl.segF, Codec<SF>::enc(f[i], T(inv_w19(i))));
    if constexpr (std::is_same<SG, Fix16>::value) {
        const RoundBits rb(node, step);
#pragma unroll
        for (int i = 0; i < 7; ++i)
            st<SG, kPolicy>(buf, s.vG, pl.offG + i * pl.segG,
                   Codec<SG>::enc_r(g[i], T(inv_w7(i)) * geo.inv_escale, rb.u16(i)));
    } else {
#pragma unroll
        for (int i = 0; i < 7; ++i)
            st<SG, kPolicy>(buf, s.vG, pl.offG + i * pl.segG, Codec<SG>::enc(g[i], T(inv_w7(i))));
    }
}

// -------------------------------------------------------------- step kernel
// floor(c / n) for c < 2^24: the float quotient is within 1/2 of the true
// one, so a single correction by one is exact.
__device__ __forceinline__ uint32_t div_small(uint32_t c, uint32_t n, float inv_n)
{
    uint32_t q = uint32_t(float(c) * inv_n);
    const int32_t r = int32_t(c) - int32_t(q * n);
    if (r < 0)
        q -= 1;
    else if (r >= int32_t(n))
        q += 1;
    return q;
}

// One thread per node, grid.z = z.  kFlat: the blocks take the plane's n^2
// nodes in storage order, so that every wavefront but the last is full for any
// n (rows of 300 nodes in blocks of 256 would leave 41 % of the lanes idle);
// otherwise a block covers (bx, by) nodes over (x, y).  kForce is the force
// model (LBMX_FORCE_*), kPolicy and kNt the policies of its stores and loads.  kThreads bounds the block: within the 128 registers that
// 1024 threads leave each, FP64 under Guo's forcing spills 36 (48^3 15.0 us against
// 8.8 us with blocks of 256, 256^3 1724 against 1230); the others fit.
constexpr int kFlatBlock = 256;
template <class St, int kForce, bool kFlat, int kThreads, int kPolicy, bool kNt>
__global__ __launch_bounds__(kThreads) void k_step(const char *__restrict__ src, char *__restrict__ dst,
                                                   Geometry<typename St::T> geo,
                                                   Rates<typename St::T> rates, float inv_n)
{
    using T = typename St::T;
    int x = blockIdx.x * blockDim.x + threadIdx.x;
    int y = blockIdx.y * blockDim.y + threadIdx.y;
    const int z = blockIdx.z;
    if (kFlat) {
        y = int(div_small(uint32_t(x), uint32_t(geo.n), inv_n));
        x -= y * geo.n;
    }
    if (x >= geo.n || y >= geo.n)
        return;
    const size_t plane = size_t(Plane<St>(uint32_t(geo.n)).bytes) * z;
    const Site s = site_in_plane<St>(geo.n, x, y, z);
    T f[19], g[7];
    pull<St, false, true, kNt>(src + plane, geo, s, y, f, g);
    collide<T, kForce>(f, g, rates);
    put<St, kPolicy>(dst + plane, s, uint32_t(x) + uint32_t(geo.n) * (uint32_t(y) + uint32_t(geo.n) * z), geo.step,
            geo, f, g);
}

// --------------------------------------------------------- state sources
// Pre-collision populations of an initial state S_0, node by node, as
// offsets (flow) and plain values (energy), in double precision.
struct SourceRest {            // f = w_i, g = w_T,i theta0
    const double *theta0;      // n^3, may be null (theta 0)
    __device__ double f(int, int) const { return 0.0; }
    __device__ double g(int i, int c) const { return theta0 ? w7(i) * theta0[c] : 0.0; }
};

// Some of the 26 population arrays of a state (numbered 0..18 flow, 19..25
// energy), each n^3 doubles: population p sits at buf + slot[p] * cells
// (slot -1: not staged).  Unstreaming population i at a node needs only
// S_i and S_ibar, so a transfer can stage the populations in opposite pairs
// and write those pairs, pass after pass, through a buffer of a few
// populations.
struct SourcePops {
    const double *buf;
    size_t cells;
    signed char slot[26];
    __device__ double f(int i, int c) const
    {
        return buf[(size_t)slot[i] * cells + c] - w19(i);
    }
    __device__ double g(int i, int c) const { return buf[(size_t)slot[19 + i] * cells + c]; }
};

// f = f^eq(rho, u) (Eq. 17) and g = w_T theta (1 + 4 e.u), whose moments are
// n^eq of Eq. (33), from node fields staged as n^3 doubles each: u, v, w, theta
// and, unless density is false (rho = 1), rho - 1.
struct SourceNodes {
    const double *buf;
    size_t cells;
    bool density;
    __device__ double f(int i, int c) const
    {
        const double vel[3] = {buf[c], buf[cells + c], buf[2 * cells + c]};
        const int e[3] = {ex19(i), ey19(i), ez19(i)};
        double eu = e[0] * vel[0] + e[1] * vel[1] + e[2] * vel[2];
        double uu = vel[0] * vel[0] + vel[1] * vel[1] + vel[2] * vel[2];
        if (!density)
            return w19(i) * (3.0 * eu + 4.5 * eu * eu - 1.5 * uu);
        const double dr = buf[4 * cells + c];
        return w19(i) * (dr + (1.0 + dr) * (3.0 * eu + 4.5 * eu * eu - 1.5 * uu));
    }
    __device__ double g(int i, int c) const
    {
        const double vel[3] = {buf[c], buf[cells + c], buf[2 * cells + c]}, t = buf[3 * cells + c];
        const int e[3] = {i == 1 ? 1 : (i == 2 ? -1 : 0), i == 3 ? 1 : (i == 4 ? -1 : 0),
                          i == 5 ? 1 : (i == 6 ? -1 : 0)};
        return w7(i) * t * (1.0 + 4.0 * (e[0] * vel[0] + e[1] * vel[1] + e[2] * vel[2]));
    }
};

// Velocity / temperature (and optionally density) fields sampled
// trilinearly from a node-centred src_n^3 grid of element type E (FP32
// fields from a caller or a network, FP64 fields of another cavity).  The
// sampled velocities are multiplied by vscale (1 keeps them bitwise) and
// rho - 1 by vscale^2 (hydrostatic and dynamic pressure go with u_c^2).
template <class E>
struct SourceFields {
    const E *u, *v, *w, *th;
    int src_n, n;
    E vscale;
    const E *rho;  // density field, or null for rho = 1
    __device__ E sample(const E *a, int x, int y, int z) const
    {
        const E s = E(src_n) / E(n);
        E p[3] = {(x + E(0.5)) * s - E(0.5), (y + E(0.5)) * s - E(0.5), (z + E(0.5)) * s - E(0.5)};
        int i0[3];
        E fr[3];
        for (int d = 0; d < 3; ++d) {
            E q = fmin(fmax(p[d], E(0)), E(src_n - 1));
            int k = min(int(floor(q)), src_n - 2 < 0 ? 0 : src_n - 2);
            i0[d] = k;
            fr[d] = q - E(k);
        }
        auto at = [&](int dx, int dy, int dz) {
            int xx = min(i0[0] + dx, src_n - 1), yy = min(i0[1] + dy, src_n - 1),
                zz = min(i0[2] + dz, src_n - 1);
            return a[xx + (size_t)src_n * (yy + (size_t)src_n * zz)];
        };
        E c00 = at(0, 0, 0) * (1 - fr[0]) + at(1, 0, 0) * fr[0];
        E c10 = at(0, 1, 0) * (1 - fr[0]) + at(1, 1, 0) * fr[0];
        E c01 = at(0, 0, 1) * (1 - fr[0]) + at(1, 0, 1) * fr[0];
        E c11 = at(0, 1, 1) * (1 - fr[0]) + at(1, 1, 1) * fr[0];
        E c0 = c00 * (1 - fr[1]) + c10 * fr[1];
        E c1 = c01 * (1 - fr[1]) + c11 * fr[1];
        return c0 * (1 - fr[2]) + c1 * fr[2];
    }
    __device__ void node(int c, double *vel, double &theta) const
    {
        int x = c % n, y = (c / n) % n, z = c / (n * n);
        vel[0] = sample(u, x, y, z) * vscale;
        vel[1] = sample(v, x, y, z) * vscale;
        vel[2] = sample(w, x, y, z) * vscale;
        theta = sample(th, x, y, z);
    }
    __device__ bool density() const { return rho != nullptr; }
    __device__ double excess(int c) const  // rho - 1
    {
        const int x = c % n, y = (c / n) % n, z = c / (n * n);
        return (double(sample(rho, x, y, z)) - 1.0) * double(vscale) * double(vscale);
    }
};

// Fields combined from two node-centred grids (FP64 fields of two other
// cavities): u = wa u_a + wb u_b, theta = wa theta_a + wb theta_b and
// rho - 1 = wa (rho_a - 1) + wb (rho_b - 1), each sampled trilinearly as by
// SourceFields (velocities scaled by its vscale, density variations by
// vscale^2).
struct SourceTwoFields {
    SourceFields<double> a, b;  // with density fields
    double wa, wb;
    __device__ void node(int c, double *vel, double &theta) const
    {
        double va[3], vb[3], ta, tb;
        a.node(c, va, ta);
        b.node(c, vb, tb);
        for (int d = 0; d < 3; ++d)
            vel[d] = wa * va[d] + wb * vb[d];
        theta = wa * ta + wb * tb;
    }
    __device__ bool density() const { return true; }
    __device__ double excess(int c) const
    {
        const int x = c % a.n, y = (c / a.n) % a.n, z = c / (a.n * a.n);
        return wa * (a.sample(a.rho, x, y, z) - 1.0) * a.vscale * a.vscale +
               wb * (b.sample(b.rho, x, y, z) - 1.0) * b.vscale * b.vscale;
    }
};

// The fields of src at every node of plane blockIdx.y, as SourceNodes reads them.
// Once per node, where each of the 26 populations would sample its own target
// node: 192^3 from 96^3 3.43 ms in one pass, 0.77 in two (0.15 here, bound by the
// FP64 interpolation; 0.54 in k_unstream, by the reads of 26 targets from cache).
template <typename Src>
__global__ __launch_bounds__(256) void k_sample(double *__restrict__ out, int n, size_t cells, Src src)
{
    const int cp = blockIdx.x * blockDim.x + threadIdx.x;
    if (cp >= n * n)
        return;
    const int c = cp + n * n * int(blockIdx.y);
    double vel[3], t;
    src.node(c, vel, t);
    for (int d = 0; d < 3; ++d)
        out[d * cells + c] = vel[d];
    out[3 * cells + c] = t;
    if (src.density())
        out[4 * cells + c] = src.excess(c);
}

// "Unstream": write the post-collision lattice P whose pull reproduces S.
// For population i at node y: if y + e_i is inside, P_i(y) = S_i(y + e_i);
// otherwise P_i(y) is the value that the wall turns into S_ibar(y).  Only
// the populations whose bit is set in `mask` (bit p: population p, flow
// 0..18, energy 19..25) are written.
// One thread per node of plane blockIdx.y.
template <class St, typename Src>
__global__ __launch_bounds__(256) void k_unstream(char *__restrict__ dst,
                                                  Geometry<typename St::T> geo, Src srcS,
                                                  uint32_t mask)
{
    using T = typename St::T;
    using SF = typename St::F;
    using SG = typename St::G;
    const int n = geo.n;
    const int cp = blockIdx.x * blockDim.x + threadIdx.x;
    if (cp >= n * n)
        return;
    const int x = cp % n, y = cp / n, z = blockIdx.y;
    const int c = x + n * (y + n * z);
    const Plane<St> pl{uint32_t(geo.n)};
    const Buffer plane = make_buffer(dst + size_t(pl.bytes) * z);
    for (int i = 0; i < 19; ++i) {
        if (!((mask >> i) & 1u))
            continue;
        const int tx = x + ex19(i), ty = y + ey19(i), tz = z + ez19(i);
        const bool in = tx >= 0 && tx < n && ty >= 0 && ty < n && tz >= 0 && tz < n;
        double v = in ? srcS.f(i, tx + n * (ty + n * tz)) : srcS.f(opp19(i), c);
        st<SF, kFar>(plane, uint32_t(cp) * pl.bF, i * pl.segF, Codec<SF>::enc(T(v), T(inv_w19(i))));
    }
    const double th_lin = double(geo.theta_hot) +
                          double(geo.theta_cold - geo.theta_hot) * (y + 0.5) / n;
    const int gx[7] = {0, 1, -1, 0, 0, 0, 0}, gy[7] = {0, 0, 0, 1, -1, 0, 0},
              gz[7] = {0, 0, 0, 0, 0, 1, -1}, go[7] = {0, 2, 1, 4, 3, 6, 5};
    for (int i = 0; i < 7; ++i) {
        if (!((mask >> (19 + i)) & 1u))
            continue;
        const int tx = x + gx[i], ty = y + gy[i], tz = z + gz[i];
        double v;
        if (tx >= 0 && tx < n && ty >= 0 && ty < n && tz >= 0 && tz < n) {
            v = srcS.g(i, tx + n * (ty + n * tz));
        } else {
            const double s_in = srcS.g(go[i], c);
            bool dir;
            double tw = 0.0;
            if (ty < 0) { dir = true; tw = double(geo.theta_hot); }
            else if (ty >= n) { dir = true; tw = double(geo.theta_cold); }
            else if (tx < 0 || tx >= n) { dir = x_wall_dirichlet(geo.wall_type); tw = th_lin; }
            else { dir = z_wall_dirichlet(geo.wall_type); tw = th_lin; }
            // S_ibar = -P_i + 2 w theta_W (Dirichlet) or P_i (adiabatic)
            v = dir ? 2.0 * w7(go[i]) * tw - s_in : s_in;
        }
        const T inv_w = St::kScaledG ? T(inv_w7(i)) * geo.inv_escale : T(inv_w7(i));
        st<SG, kFar>(plane, uint32_t(cp) * pl.bG, pl.offG + i * pl.segG, Codec<SG>::enc(T(v), inv_w));
    }
}

// Copy a lattice from its planes into the slabs of a checkpoint file (kSave;
// slots past the last node become 0) or back.  One thread per slab slot.
template <class St, bool kSave>
__global__ __launch_bounds__(256) void k_relayout(char *__restrict__ planes, char *__restrict__ slabs, int n,
                                                  size_t slots)
{
    using RF = typename Codec<typename St::F>::Raw;
    using RG = typename Codec<typename St::G>::Raw;
    constexpr int L = St::kSlabShift;
    constexpr size_t segF = sizeof(RF) << L, segG = sizeof(RG) << L, slab = 19 * segF + 7 * segG;
    const size_t c = size_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (c >= slots)
        return;
    const size_t nn = size_t(n) * n, slot = c & ((size_t(1) << L) - 1);
    const bool node = c < nn * n;
    const Plane<St> pl{uint32_t(n)};
    char *const sl = slabs + (c >> L) * slab;
    char *const pp = planes + c / nn * pl.bytes;
    const size_t cp = c % nn;
    auto move = [&](auto *file, auto *lat) {
        if (kSave)
            *file = node ? *lat : 0;
        else if (node)
            *lat = *file;
    };
    for (int i = 0; i < 19; ++i)
        move(reinterpret_cast<RF *>(sl + i * segF) + slot, reinterpret_cast<RF *>(pp + size_t(i) * pl.segF) + cp);
    for (int i = 0; i < 7; ++i)
        move(reinterpret_cast<RG *>(sl + 19 * segF + i * segG) + slot,
             reinterpret_cast<RG *>(pp + pl.offG + size_t(i) * pl.segG) + cp);
}

// ------------------------------------------------------------ read kernels
// Macroscopic fields at time t: rho, u = j / rho, theta (double outputs).
// Guo's forcing reports u_z = j_z / rho + vshift (theta - theta_ref) with
// vshift = g beta / 2 (the half-force velocity); vshift = 0 otherwise.
template <class St>
__global__ __launch_bounds__(256) void k_macro(const char *__restrict__ src,
                                               Geometry<typename St::T> geo, double vshift,
                                               double theta_ref, double *rho, double *ux,
                                               double *uy, double *uz, double *theta)
{
    using T = typename St::T;
    const int n = geo.n;
    const int cp = blockIdx.x * blockDim.x + threadIdx.x;
    if (cp >= n * n)
        return;
    const int x = cp % n, y = cp / n, z = blockIdx.y;
    const size_t c = size_t(cp) + size_t(n) * n * z;
    T f[19], g[7];
    pull<St, false>(src + size_t(Plane<St>(uint32_t(geo.n)).bytes) * z, geo, site_in_plane<St>(n, x, y, z), y, f,
                    g);
    double dr = 0.0, j[3] = {0.0, 0.0, 0.0}, th = 0.0;
    for (int i = 0; i < 19; ++i) {
        dr += double(f[i]);
        j[0] += ex19(i) * double(f[i]);
        j[1] += ey19(i) * double(f[i]);
        j[2] += ez19(i) * double(f[i]);
    }
    for (int i = 0; i < 7; ++i)
        th += double(g[i]);
    const double r = 1.0 + dr;
    if (rho) rho[c] = r;
    if (ux) ux[c] = j[0] / r;
    if (uy) uy[c] = j[1] / r;
    if (uz) uz[c] = vshift != 0.0 ? j[2] / r + vshift * (th - theta_ref) : j[2] / r;
    if (theta) theta[c] = th;
}

// Populations first .. first + count - 1 (flow 0..18, energy 19..25) at
// time t as plain doubles: out[(p - first) * n^3 + c].
template <class St>
__global__ __launch_bounds__(256) void k_pops(const char *__restrict__ src,
                                              Geometry<typename St::T> geo, int first, int count,
                                              double *out)
{
    using T = typename St::T;
    const int n = geo.n;
    const int cp = blockIdx.x * blockDim.x + threadIdx.x;
    if (cp >= n * n)
        return;
    const int x = cp % n, y = cp / n, z = blockIdx.y;
    const size_t c = size_t(cp) + size_t(n) * n * z;
    T f[19], g[7];
    pull<St, false>(src + size_t(Plane<St>(uint32_t(geo.n)).bytes) * z, geo, site_in_plane<St>(n, x, y, z), y, f,
                    g);
    const size_t cells = size_t(n) * n * n;
    for (int k = 0; k < count; ++k) {
        const int p = first + k;
        out[(size_t)k * cells + c] = p < 19 ? w19(p) + double(f[p]) : double(g[p - 19]);
    }
}

// --------------------------------------------------------- Nusselt number
// Wavefront-wide reductions (64 lanes on CDNA).
__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
        v += __shfl_xor(v, o, 64);
    return v;
}
__device__ __forceinline__ double wave_max(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
        v = fmax(v, __shfl_xor(v, o, 64));
    return v;
}

// Combine 4 per-lane accumulators (sum, line, max, bad) across the block:
// wavefront shuffles, then the first lane of each wave through LDS.  The
// block-wide result is valid in thread 0.
__device__ __forceinline__ void block_reduce4(double &sum, double &line, double &mx, double &bad)
{
    __shared__ double red[4][16];
    sum = wave_sum(sum);
    line = wave_sum(line);
    mx = wave_max(mx);
    bad = wave_sum(bad);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0) {
        red[0][wv] = sum;
        red[1][wv] = line;
        red[2][wv] = mx;
        red[3][wv] = bad;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const int nw = (blockDim.x + 63) >> 6;
        double s = 0.0, l = 0.0, m = -1.0e300, b = 0.0;
        for (int k = 0; k < nw; ++k) {
            s += red[0][k];
            l += red[1][k];
            m = fmax(m, red[2][k]);
            b += red[3][k];
        }
        sum = s;
        line = l;
        mx = m;
        bad = b;
    }
}

// One block per z row of the hot wall (y = 0).  Local Nu (Eq. 39) from the
// wall-adjacent nodes, by stencil (LBMX_NU_*):
//   0  second order, dtheta/dy = (9 th0 - th1 - 8 th_w)/3;
//   1  first order, dtheta/dy = 2 (th0 - th_w);
//   2  energy crossing the wall links, q = 2 (g_+y - th_w / 8), as -q / D_yy
//      (g_+y at the wall node is the population that came from the wall).
// partial[z] = {sum over x, X = 0.5 line contribution, max, non-finite count}.
template <class St>
__global__ __launch_bounds__(256) void k_nu_rows(const char *__restrict__ src,
                                                 Geometry<typename St::T> geo, double theta_hot,
                                                 int stencil, double d_yy, double *partial,
                                                 double *map)
{
    using T = typename St::T;
    const int n = geo.n;
    const int z = blockIdx.x;
    const char *const plane = src + size_t(Plane<St>(uint32_t(geo.n)).bytes) * z;
    double sum = 0.0, line = 0.0, mx = -1.0e300, bad = 0.0;
    for (int x = threadIdx.x; x < n; x += blockDim.x) {
        T f[19], g0[7], g1[7];
        pull<St, false>(plane, geo, site_in_plane<St>(n, x, 0, z), 0, f, g0);
        double th0 = 0.0, th1 = 0.0;
        for (int i = 0; i < 7; ++i)
            th0 += double(g0[i]);
        double nu;
        if (stencil == 1) {
            nu = -double(n) * 2.0 * (th0 - theta_hot);
        } else if (stencil == 2) {
            nu = double(n) * 2.0 * (double(g0[3]) - 0.125 * theta_hot) / d_yy;
        } else {
            pull<St, false>(plane, geo, site_in_plane<St>(n, x, 1, z), 1, f, g1);
            for (int i = 0; i < 7; ++i)
                th1 += double(g1[i]);
            nu = -double(n) * (9.0 * th0 - th1 - 8.0 * theta_hot) / 3.0;
        }
        if (map)
            map[x + (size_t)n * z] = nu;
        if (!isfinite(nu)) {
            bad += 1.0;
            continue;
        }
        sum += nu;
        mx = fmax(mx, nu);
        if (n & 1) {
            if (x == n / 2) line += nu;
        } else if (x == n / 2 - 1 || x == n / 2) {
            line += 0.5 * nu;
        }
    }
    block_reduce4(sum, line, mx, bad);
    if (threadIdx.x == 0) {
        partial[4 * z + 0] = sum;
        partial[4 * z + 1] = line;
        partial[4 * z + 2] = mx;
        partial[4 * z + 3] = bad;
    }
}

// Combine the per-row partials in a fixed order: out = {Nu_3D, Nu_2D, Nu_max, bad}.
// (A template only so that every translation unit may include this header.)
template <int kUnused = 0>
__global__ __launch_bounds__(256) void k_nu_final(const double *partial, int n, double *out)
{
    double sum = 0.0, line = 0.0, mx = -1.0e300, bad = 0.0;
    for (int z = threadIdx.x; z < n; z += blockDim.x) {
        sum += partial[4 * z + 0];
        line += partial[4 * z + 1];
        mx = fmax(mx, partial[4 * z + 2]);
        bad += partial[4 * z + 3];
    }
    block_reduce4(sum, line, mx, bad);
    if (threadIdx.x == 0) {
        out[0] = sum / (double(n) * double(n));  // Eq. (40), midpoint rule
        out[1] = line / double(n);               // Eq. (41), midpoint rule
        out[2] = mx;
        out[3] = bad;
    }
}

}  // namespace lbmx
