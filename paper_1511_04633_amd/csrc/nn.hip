// nn.hip -- hand-written BF16 / FP32 kernels of the 3-D convolutional U-Net
// that predicts steady cavity fields from (Ra, wall type) and warm-starts
// the lattice Boltzmann solve.
//
// Tensors: activations are channel-last BF16, [B][D][H][W][C] with C a
// multiple of 16; 3x3x3 convolution weights are BF16 [Co][27][Ci] with tap
// t = (kz*3 + ky)*3 + kx at offset (kx-1, ky-1, kz-1); biases, weight
// gradients, Adam state and master weights are FP32.
//
// Convolution = implicit GEMM on the matrix cores: out[p][co] =
// sum_{tap, ci} W[co][tap][ci] in[p + off(tap)][ci] with M = co, N = voxels,
// K = (tap, ci), FP32 accumulation.  Both convolution kernels run on
// v_mfma_f32_16x16x32_bf16 (gfx950) over bricks of voxels staged in LDS, so that
// each staged element serves all 27 taps, in an order in which the blocks of one
// XCD work on neighbours:
//   - forward (and the data gradient, the same convolution of the output
//     gradient with the flipped, transposed weights W'[ci][26-tap][co] =
//     W[co][tap][ci]): a block walks bricks of 16 x 4 x 4 or 16 x 4 x 8 voxels
//     (brick_walk) and stages a brick's input with a one-voxel halo and the
//     weights of all taps per 16 input channels, channel-last; K = 32
//     covers two taps of the 16 channels; the epilogue can apply SiLU, its
//     derivative, a channel split or the squared-error loss; the input can be
//     a decoder's upsampled-and-concatenated tensor read in place; details
//     at k_conv_fwd;
//   - weight gradient: a block owns one (output-channel tile, input-channel
//     tile) pair and streams a range of chunks of 16 x 8 x 4 voxels down columns,
//     bringing output gradient and input halo into LDS as they lie in memory;
//     transposing LDS reads give the operands, K = 32 covering two rows of voxels;
//     the bias gradient is one
//     more MFMA against ones; the block's sums are added to the global gradient
//     atomically; details at k_conv_wgrad.
// MFMA operand layout of v_mfma_f32_16x16x32_bf16 (checked on the device):
// lane l holds A[l%16][8(l/16) .. 8(l/16)+7] and B[8(l/16) .. 8(l/16)+7][l%16]
// and gets D[4(l/16)+j][l%16], j < 4.
#include <hip/hip_bf16.h>
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "host.hpp"

using namespace lbmx::host;

namespace {

typedef short s4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));
using bf = unsigned short;  // BF16 bits

__device__ __forceinline__ float bf2f(bf h) { return __uint_as_float(uint32_t(h) << 16); }
__device__ __forceinline__ bf f2bf(float f) { return __bfloat16_as_ushort(__float2bfloat16(f)); }

// SiLU a = z sigma(z) and its backward dz = da sigma(z) (1 + z (1 - sigma(z))),
// shared by the elementwise kernels and the convolution epilogues so that the
// fused and the separate paths compute the same expression.  sigma uses the
// hardware reciprocal (v_rcp_f32, about 1 ulp of FP32) instead of an IEEE
// division: the results are rounded to BF16 (8-bit significand), and the
// division's scale / fixup sequence dominated the convolution epilogues.
__device__ __forceinline__ float sigmoid_f(float v) { return __builtin_amdgcn_rcpf(1.f + __expf(-v)); }
__device__ __forceinline__ float silu_f(float v) { return v * sigmoid_f(v); }
__device__ __forceinline__ float silu_grad_f(float ga, float v)
{
    const float sg = sigmoid_f(v);
    return ga * sg * (1.f + v * (1.f - sg));
}

struct Dims {
    int B, D, H, W;  // batch and spatial extent
    int Ci, Co;      // channels (multiples of 16)
};

// ------------------------------------------------------------- convolution
// out[p][co] = bias[co] + sum_{tap, ci} W[co][tap][ci] in[p + off(tap)][ci].
//
// A block owns NCO output channel tiles of 16 (blockIdx.y selects the group)
// and walks bricks of 16 x 4 x 4 voxels in the XCD-aware order of
// brick_walk.  Per round of 16 input channels it stages in LDS, channel-last:
//   x: the brick's input plus a one-voxel halo (18 x 6 x 6 voxels, or 18 x 6 x
//      10), so the MFMA operand "8 consecutive input channels of the voxel at
//      this tap" is one aligned 16-byte read for any tap;
//   w: the weights of the block's output channels for all 27 taps, plus a
//      28th tap of zeros.
// Both come from memory straight into LDS (buffer loads to LDS; voxels outside
// the volume are out of the buffer's range and arrive as zeros).  A row (16
// channels, 32 bytes) holds its two 8-channel halves swapped when bit 2 of its x
// (halo x for x, output channel for w) is set, by each lane fetching the half that
// belongs at its place: the 8 lanes of a 16-byte LDS read phase then cover all
// banks.  The products run on v_mfma_f32_16x16x32_bf16 (gfx950; lane layout
// checked on the device): its K = 32 covers two taps of the round's 16 channels
// (lanes 0-31 tap 2p, lanes 32-63 tap 2p + 1, p < 14).  The 28th tap has zero
// weights and reads its input operand from a zeroed LDS block, so non-finite
// inputs cannot leak into it.  A wave computes 4 rows of 16 voxels (8 in two
// planes): a weight operand serves all of them, and an input operand the NCO
// channel tiles and every (row, tap pair) that it lies at (TapPairs), which
// leaves 50 (39) of 56 input reads per 4 rows.  Each lane ends with 4 consecutive
// output channels of one voxel and stores them together.
// Per round: wait for the tiles, products, request the next round's tiles into
// the same place, and finish and store a brick's results while they travel: the
// wait counts off the stores, which are one instruction per row and tile for
// every wave, excluded lanes by their offset.  The other blocks of the CU (4 with
// one channel tile) fill the waits.
// Bound by LDS reads (15 of 29 us at 64^3 16 -> 16 before they were shared) and,
// with the SiLU beside z, by the stores (18 us alone).  Batch 4, us, tiles through
// registers -> here: 64^3 16 -> 16 35 -> 26.5, 48 -> 16 72 -> 53, 32^3 96 -> 32 32 ->
// 28.5, 16^3 64 -> 64 12.2 -> 10.8, 8^3 96 -> 96 13.4 -> 10.4; data gradients 64^3 16 ->
// 16 38 -> 30, 16 -> 48 74 -> 47, 32^3 32 -> 96 39 -> 28.  Two buffers and two blocks per
// CU instead: 34.
typedef __bf16 bf8v __attribute__((ext_vector_type(8)));
constexpr int FC_X = 16, FC_Y = 4;                  // brick: 16 x 4 x 4 RZ voxels
constexpr int FC_HX = FC_X + 2, FC_HY = FC_Y + 2;
constexpr int FC_ROW = FC_HX * 16;                  // elements of a halo row
constexpr int FC_THREADS = 256;                     // block size (the launcher's)
constexpr int FC_ZERO = 3 * FC_ROW + 16;            // zero block: the padding tap's 4 row reads
constexpr int FC_WLOADS(int nco) { return (27 * nco * 32 + 63) / 64; }  // wave loads of a weight tile
constexpr int FC_WITERS(int nco) { return (FC_WLOADS(nco) + 3) / 4; }   // per wave

// element offset of half `part` of row `row` whose swizzle bit is `sx`
__device__ __forceinline__ int fc_slot(int row, int part, int sx)
{
    return row * 16 + 8 * (part ^ ((sx >> 2) & 1));
}

// floor(j / n) for 0 <= j < 2^24 from the float reciprocal: the float
// quotient is within one of the true one, so one correction is exact.
__device__ __forceinline__ int fdiv_small(int j, int n, float inv_n)
{
    int q = int(float(j) * inv_n);
    const int r = j - q * n;
    if (r < 0)
        --q;
    else if (r >= n)
        ++q;
    return q;
}

// Brick j of a [B][nbz][nby][nbx] grid of bricks (x fastest): batch index
// and the brick's first voxel (brick counts are below 2^23).
struct BrickGrid {
    int nbx, nby, nbz;
    float inx, iny, inz;
    __device__ BrickGrid(int x, int y, int z)
        : nbx(x), nby(y), nbz(z), inx(1.f / x), iny(1.f / y), inz(1.f / z)
    {
    }
    __device__ __forceinline__ void at(int j, int sx, int sy, int sz, int &b, int &x0, int &y0, int &z0) const
    {
        const int r1 = fdiv_small(j, nbx, inx), r2 = fdiv_small(r1, nby, iny);
        b = fdiv_small(r2, nbz, inz);
        x0 = (j - r1 * nbx) * sx, y0 = (r1 - r2 * nby) * sy, z0 = (r2 - b * nbz) * sz;
    }
};

// The bricks a block walks.  Workgroup i runs on XCD i mod 8 (for a grid
// whose x extent is a multiple of 8 this is blockIdx.x mod 8), and each XCD
// has its own L2; a block takes bricks first, first + stride, ... of its
// XCD's contiguous eighth of all bricks, so the bricks in flight on one XCD
// are neighbours whose halos overlap and are read through one L2.  Other
// grids take bricks blockIdx.x, blockIdx.x + gridDim.x, ...
struct BrickWalk {
    int first, stride, count;
};

__device__ __forceinline__ BrickWalk brick_walk(int nbricks)
{
    const int G = int(gridDim.x), bx = int(blockIdx.x);
    BrickWalk r;
    if (G % 8 == 0) {
        const int xcd = bx % 8, S = G / 8;
        const int lo = int((long long)xcd * nbricks / 8), hi = int((long long)(xcd + 1) * nbricks / 8);
        r.first = lo + bx / 8;
        r.stride = S;
        r.count = r.first < hi ? (hi - 1 - r.first) / S + 1 : 0;
    } else {
        r.first = bx;
        r.stride = G;
        r.count = bx < nbricks ? (nbricks - 1 - bx) / G + 1 : 0;
    }
    return r;
}

// The convolution input: channel-last in[B][D][H][W][Ci], or for a decoder
// layer the concatenation of the nearest x2 upsampling of low
// [B][D/2][H/2][W/2][cu] (channels 0 .. cu-1) with skip [B][D][H][W][Ci-cu]
// (channels cu .. Ci-1), read in place: a 16-channel round or tile lies in
// one of the two (cu is a multiple of 16), so the choice is uniform.
struct ConvIn {
    const bf *in;   // the input, or the skip part
    const bf *low;  // null for a plain input
    int cu;         // channels taken from low (0 for a plain input)
};

// Epilogue options of a BF16 output (all null / 0 for the plain convolution):
//   act:   also write a = silu(z) beside z = conv + bias (forward layers);
//   gate:  write bf16(bf16(conv) * silu'(gate)) instead of the convolution:
//          the data gradient of a layer times the SiLU derivative at the
//          previous layer's pre-activation gate, i.e. that layer's dL/dz;
//   out2, split: output channels >= split go to out2 (Co - split channels per
//          voxel), the others to out (split per voxel): the two halves of a
//          concatenated input's gradient.
struct Epilogue {
    bf *act;
    const bf *gate;
    bf *out2;
    int split;
};

// The squared-error loss fused into a head convolution (k_conv_fwd with
// LOSS): z = conv + bias stays FP32 in registers; for channels c < K,
// e = z - target[p][c], grad[p][c] = bf16(2 e scale), 0 for c >= K; each
// block writes the sum of its e^2 to partial[block] and block 0 clears
// partial[blocks .. npartial); out (FP32 [.][Co]) receives z if not null.
struct LossEp {
    const float *target;
    int K;
    float scale;
    bf *grad;
    double *partial;
    int npartial;
};

// 16 bytes per lane from `offset` of base into lds + 16 lane; zeros where the
// offset is kOutside.  kDirect: straight into LDS (wait_loads), for a 16-byte
// aligned base; the offset is in units of 1 / load_units elements.
constexpr uint32_t kRange = 0xffffff00u, kOutside = 0xffffffffu;
constexpr uint32_t load_units(bool direct) { return direct ? 2 : 1; }  // bytes, which must stay below kRange
template <bool kDirect>
__device__ __forceinline__ void load_to_lds(const bf *base, bf *lds, int lane, uint32_t offset)
{
    if constexpr (kDirect) {
        using L = __attribute__((address_space(3))) void;
        const auto r = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf *>(base), short(0), int(kRange), 0x00020000);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (L *)lds, 16, offset, 0, 0, 0);
    } else {
        uint4 v = make_uint4(0, 0, 0, 0);
        if (offset != kOutside)
            __builtin_memcpy(&v, base + offset, 16);
        *reinterpret_cast<uint4 *>(lds + lane * 8) = v;
    }
}

// Which positions of a tile lie inside the volume: a position's x, y, z are a
// byte each with the top bit set (tile_pos), and one subtraction from either end
// of the valid range keeps the top bits of the bytes in it.  Five instructions
// per position, where the comparisons of positions found anew by division took
// about 25, a third of the arithmetic of a round at the volume's faces (62 % of
// the bricks of 64^3).
constexpr uint32_t kTops = 0x808080u;
__device__ __forceinline__ uint32_t tile_pos(int x, int y, int z) { return kTops | uint32_t(x | y << 8 | z << 16); }
struct TileRange {
    uint32_t lo, hi;
    // positions from (lx, ly, lz) to (hx, hy, hz), all non-negative; none if hz < 0
    __device__ __forceinline__ TileRange(int lx, int ly, int lz, int hx, int hy, int hz)
        : lo(uint32_t(lx | ly << 8 | (hz < 0 ? 127 : lz) << 16)),
          hi(2 * kTops + uint32_t(min(hx, 127) | min(hy, 127) << 8 | max(min(hz, 127), 0) << 16))
    {
    }
    __device__ __forceinline__ bool has(uint32_t pos) const { return ((pos - lo) & (hi - pos) & kTops) == kTops; }
};
// Wait until no more than n of this wave's memory operations are on their way
// (vmcnt n): its loads to LDS before the last n.
template <int n = 0>
__device__ __forceinline__ void wait_loads()
{
    static_assert(n < 64);
    __builtin_amdgcn_s_waitcnt(0x0f70 | (n & 15) | (n >> 4 << 14));
}

// A barrier that orders LDS accesses but leaves loads to LDS on their way, where
// __syncthreads would wait for them (vmcnt 0).
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt 0: this wave's reads of LDS are done
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

typedef uint32_t v2u __attribute__((ext_vector_type(2)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
__device__ __forceinline__ auto buffer_of(const void *base, int range)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), short(0), range, 0x00020000);
}
// A lane's 8 or 16 bytes at a byte offset of base; nothing (zeros) where the
// offset or the range (0 or kRange) excludes it.  kDirect (an aligned base): one
// instruction for the whole wave, whichever lanes are excluded.
template <bool kDirect, class V>
__device__ __forceinline__ void store_vec(void *base, int range, V v, uint32_t offset)
{
    if constexpr (!kDirect) {
        if (range && offset != kOutside)
            __builtin_memcpy(static_cast<char *>(base) + offset, &v, sizeof v);
    } else if constexpr (sizeof(V) == 8) {
        __builtin_amdgcn_raw_buffer_store_b64(v, buffer_of(base, range), offset, 0, 0);
    } else {
        __builtin_amdgcn_raw_buffer_store_b128(v, buffer_of(base, range), offset, 0, 0);
    }
}
template <bool kDirect>
__device__ __forceinline__ v2u load_vec(const void *base, int range, uint32_t offset)
{
    v2u v{0, 0};
    if constexpr (kDirect)
        v = __builtin_amdgcn_raw_buffer_load_b64(buffer_of(base, range), offset, 0, 0);
    else if (range && offset != kOutside)
        __builtin_memcpy(&v, static_cast<const char *>(base) + offset, sizeof v);
    return v;
}

// What the convolution writes (Epilogue and LossEp): FP32, BF16 (with or
// without split), BF16 and its SiLU, its SiLU alone, BF16 times SiLU' at gate, or
// the loss.
enum FcOut { kF32, kBf16, kAct, kSilu, kGate, kLoss };

// Occupancy is register-bound: 4 waves per SIMD for one channel tile (3 for its
// bricks of 8 planes), 2 for more and for the loss variant.
//
// KS > 1 (layers with several rounds on small grids): the block has KS
// groups of FC_THREADS threads, each with its own LDS tiles; group g takes
// rounds g, g + KS, ... of the same brick, which shortens the block's
// serial chain of rounds KS times; at the end of a brick the other groups
// add their sums into group 0's through LDS, and group 0 stores.
constexpr int fc_waves(int nco, int rz, FcOut kind, int ks)
{
    return nco == 1 && kind != kLoss && ks == 1 ? (rz == 1 ? 4 : 3) : 2;
}
template <int NCO, int RZ>
struct FcTile {
    static constexpr int Z = 4 * RZ, HZ = Z + 2;                // brick and halo extent in z
    static constexpr int PIECES = FC_HX * FC_HY * HZ * 2;       // 16-byte pieces of the input tile
    static constexpr int LOADS = (PIECES + 63) / 64;            // wave loads of 64 pieces
    static constexpr int ITERS = (LOADS + 3) / 4;               // per wave
    static constexpr int WROWS = 28 * NCO * 16;
    bf x[LOADS * 512];               // input halo
    bf zero[FC_ZERO];
    bf w[(FC_WLOADS(NCO) * 32 > WROWS ? FC_WLOADS(NCO) * 32 : WROWS) * 16];  // weights, a 28th tap of zeros
};

// The input operand of tap pair p (taps 2 p and 2 p + 1) for output row (y, z)
// of a wave is one of three kinds at halo row (y + dy, z + dz), where a row
// serves every output row and pair that it lies at:
//   kind 0: x offsets 0, 1;   kind 1: x offsets 1, 2;
//   kind 2: x offset 2, and 0 of the next row in y;
// or (pairs 4 and 13, one use each) x offset 2 of the last row of a plane's taps
// and 0 of the next plane's first (or the zeros).
struct TapPairs {
    static constexpr int kind[14] = {0, 2, 1, 0, 3, 1, 0, 2, 1, 0, 2, 1, 0, 4};
    static constexpr int dz[14] = {0, 0, 0, 0, 0, 1, 1, 1, 1, 2, 2, 2, 2, 0};
    static constexpr int dy[14] = {0, 0, 1, 2, 0, 0, 1, 1, 2, 0, 0, 1, 2, 0};
};
// The first pair that uses kind k at halo row (y, z) of a wave.
template <int RZ>
struct FirstUse {
    int pair[3][RZ + 2][FC_HY] = {};
    constexpr FirstUse()
    {
        for (int p = 13; p >= 0; --p)
            for (int z = 0; z < RZ; ++z)
                for (int y = 0; y < 4; ++y)
                    if (TapPairs::kind[p] < 3)
                        pair[TapPairs::kind[p]][z + TapPairs::dz[p]][y + TapPairs::dy[p]] = p;
    }
};

template <int NCO, int RZ, FcOut kOut, int KS, bool kDirect>
__global__ __launch_bounds__(FC_THREADS * KS) __attribute__((amdgpu_waves_per_eu(fc_waves(NCO, RZ, kOut, KS)))) void
k_conv_fwd(ConvIn src, const bf *__restrict__ w, const float *__restrict__ bias, void *__restrict__ out,
           Dims d, int nbx, int nby, int nbz, Epilogue ep, LossEp ls)
{
    using Tile = FcTile<NCO, RZ>;
    constexpr int kWaves = fc_waves(NCO, RZ, kOut, KS), NR4 = 4 * RZ;  // rows of a wave
    constexpr bool kAhead = kWaves <= 2;
    constexpr int NBUF = KS > 1 ? 2 : 1;
    __shared__ __attribute__((aligned(16))) Tile tiles[KS][NBUF];
    static_assert(KS == 1 || NR4 * NCO * FC_THREADS * sizeof(f4) <= sizeof(tiles[0][0].x), "room for a group's sums");
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
    const int tid = int(threadIdx.x) % FC_THREADS, kg = wave / 4;
    const int Ci = d.Ci, Co = d.Co;
    const int lane = tid & 63, wv = wave % 4;
    const int col = lane & 15, kq = lane >> 4;
    const int h = kq >> 1, part = kq & 1;   // tap parity and channel half of this lane's K slice
    const int co0 = blockIdx.y * NCO * 16;
    const int nbricks = d.B * nbx * nby * nbz;
    const int R = Ci / 16;  // rounds of 16 input channels per brick
    const BrickGrid grid(nbx, nby, nbz);
    auto brick_at = [&](int j, int &bb, int &xx, int &yy, int &zz) {
        grid.at(j, FC_X, FC_Y, Tile::Z, bb, xx, yy, zz);
    };

    // This lane's pieces: wave wv runs wave loads j = wv + 4 k; piece i = 64 j +
    // lane fills 16 bytes of LDS row i / 2: the half (i % 2) ^ swizzle bit of that
    // voxel (weights: of that tap and output channel).  Offsets from the voxel
    // before the brick's first one in x, y and z (weights: from w), and positions
    // in the halo.
    constexpr uint32_t kUnits = load_units(kDirect);
    uint32_t xoff[Tile::ITERS], xpos[Tile::ITERS], woff[FC_WITERS(NCO)];
    auto halo_of = [&](int k, int &hx, int &hy, int &hz) {
        const int hv = ((wv + 4 * k) * 64 + lane) >> 1, hrow = hv / FC_HX;
        hx = hv % FC_HX, hy = hrow % FC_HY, hz = hrow / FC_HY;
    };
    auto x_offsets = [&](bool up) {  // up: voxel (x, y, z) reads low at (x/2, y/2, z/2); brick corners are even
        const int sh = up ? 1 : 0, cs = up ? src.cu : Ci - src.cu;
        const int Hi = d.H >> sh, Wi = d.W >> sh;
#pragma unroll
        for (int k = 0; k < Tile::ITERS; ++k) {
            const int hx = xpos[k] & 127, hy = (xpos[k] >> 8) & 127, hz = (xpos[k] >> 16) & 127;
            const int half = (lane & 1) ^ ((hx >> 2) & 1);
            xoff[k] = uint32_t((((hz - 1) >> sh) + 1) * Hi + ((hy - 1) >> sh) + 1) * Wi + uint32_t(((hx - 1) >> sh) + 1);
            xoff[k] = kUnits * (xoff[k] * uint32_t(cs) + uint32_t(half * 8));
        }
    };
#pragma unroll
    for (int k = 0; k < Tile::ITERS; ++k) {
        int hx, hy, hz;
        halo_of(k, hx, hy, hz);
        xpos[k] = hz < Tile::HZ ? tile_pos(hx, hy, hz) : 0u;  // the last wave load's tail is never inside
    }
    bool up_now = src.cu > 0;
    x_offsets(up_now);
#pragma unroll
    for (int k = 0; k < FC_WITERS(NCO); ++k) {
        const int row = ((wv + 4 * k) * 64 + lane) >> 1, tap = row / (NCO * 16), co = row % (NCO * 16);
        const int half = (lane & 1) ^ ((co >> 2) & 1);
        woff[k] = tap < 27 ? kUnits * uint32_t(((co0 + co) * 27 + tap) * Ci + half * 8) : kOutside;
    }

    // With one round per brick (Ci = 16) the weights are the same for every
    // item: they are loaded with the first item of each buffer only.
    const bool w_once = R == 1;
    auto load_round = [&](int j, int c0, Tile &t, bool with_w) {
        int b, x0, y0, z0;
        brick_at(j, b, x0, y0, z0);
        const bool up = c0 < src.cu;
        if (up != up_now) {
            up_now = up;
            x_offsets(up);
        }
        const int sh = up ? 1 : 0, cs = up ? src.cu : Ci - src.cu;
        const int Di = d.D >> sh, Hi = d.H >> sh, Wi = d.W >> sh;
        const bf *const base = (up ? src.low + c0 : src.in + (c0 - src.cu)) +
                               (((long long)(b * Di + (z0 >> sh) - 1) * Hi + (y0 >> sh) - 1) * Wi + (x0 >> sh) - 1) * cs;
        const TileRange inside(x0 == 0, y0 == 0, z0 == 0, d.W - x0, d.H - y0, d.D - z0);
#pragma unroll
        for (int k = 0; k < Tile::ITERS; ++k)
            if (wv + 4 * k < Tile::LOADS)
                load_to_lds<kDirect>(base, t.x + (wv + 4 * k) * 512, lane, inside.has(xpos[k]) ? xoff[k] : kOutside);
        if (!with_w)
            return;
#pragma unroll
        for (int k = 0; k < FC_WITERS(NCO); ++k)  // [tap][co][2 x 8 ch]
            if (wv + 4 * k < FC_WLOADS(NCO))
                load_to_lds<kDirect>(w + c0, t.w + (wv + 4 * k) * 512, lane, woff[k]);
    };

    // LDS operand addresses of this lane: the weight rows of tap 2 p + h are
    // wa + (2 p NCO + j) 256 for channel tile j; the input operand of each kind
    // for the wave's first halo row is at[kind] (the others follow at FC_ROW
    // each, planes at FC_HY FC_ROW).
    Tile &t0 = tiles[kg][0];
    const bf *wa = t0.w + fc_slot(h * NCO * 16 + col, part, col);
    auto x_at = [&](int dx, int hy, int hz) {
        return t0.x + fc_slot(((wv * RZ + hz) * FC_HY + hy) * FC_HX + col + dx, part, col + dx);
    };
    const bf *at[4 + RZ];
    at[0] = x_at(h, 0, 0);
    at[1] = x_at(1 + h, 0, 0);
    at[2] = h ? x_at(0, 1, 0) : x_at(2, 0, 0);
    at[3] = h ? x_at(0, 0, 1) : x_at(2, 2, 0);
#pragma unroll
    for (int rz = 0; rz < RZ; ++rz)
        at[4 + rz] = h ? t0.zero : x_at(2, 2, rz + 2);

    f4 acc[NR4][NCO];
#pragma unroll
    for (int rr = 0; rr < NR4; ++rr)
#pragma unroll
        for (int j = 0; j < NCO; ++j)
            acc[rr][j] = f4{0.f, 0.f, 0.f, 0.f};
    double sq = 0.0;  // kLoss: this lane's sum of squared errors
    f4 bj[NCO];       // without a bias -0, which leaves every sum as it is
#pragma unroll
    for (int j = 0; j < NCO; ++j)
#pragma unroll
        for (int k = 0; k < 4; ++k)
            bj[j][k] = bias ? bias[co0 + j * 16 + kq * 4 + k] : -0.f;

    for (int q = 0; q < NBUF; ++q) {
        if (FC_WLOADS(NCO) * 512 <= 27 * NCO * 256)  // else the last wave load writes zeros there
            for (int i = tid; i < NCO * 16 * 16 / 8; i += FC_THREADS)
                reinterpret_cast<uint4 *>(tiles[kg][q].w + 27 * NCO * 16 * 16)[i] = make_uint4(0, 0, 0, 0);
        else
            for (int i = tid + FC_WLOADS(NCO) * 64 - 27 * NCO * 32; i < NCO * 16 * 16 / 8; i += FC_THREADS)
                reinterpret_cast<uint4 *>(tiles[kg][q].w + 27 * NCO * 16 * 16)[i] = make_uint4(0, 0, 0, 0);
        for (int i = tid; i < FC_ZERO / 8; i += FC_THREADS)
            reinterpret_cast<uint4 *>(tiles[kg][q].zero)[i] = make_uint4(0, 0, 0, 0);
    }
    const BrickWalk bw = brick_walk(nbricks);
    const int NR = (R + KS - 1) / KS;  // steps per brick; group kg takes round kg + KS step
    const int nitems = bw.count * NR;  // (brick, step) pairs of this block
    auto round_of = [&](int it) { return kg + KS * (it % NR); };
    auto load_item = [&](int it) {
        if (it < nitems && round_of(it) < R)
            load_round(bw.first + (it / NR) * bw.stride, round_of(it) * 16, tiles[kg][NBUF > 1 ? it & 1 : 0],
                       !w_once || it < NBUF);
    };
    load_item(0);
    wait_loads();
    for (int item = 0; item < nitems; ++item) {
        const int step = item % NR, round = round_of(item);
        const bool active = round < R;  // false for a group left without a round (R % KS != 0)
        const bool last = step + 1 == NR;
        int b, x0, y0, z0;
        brick_at(bw.first + (item / NR) * bw.stride, b, x0, y0, z0);
        // The wave's rows of this brick: voxel row0(rr) + col; rows outside the volume have an empty range, lanes outside it an
        // offset out of range.
        const int z = z0 + wv * RZ;
        const bool xin = x0 + col < d.W;
        auto row0 = [&](int rr) {
            return ((long long)(b * d.D + z + rr / 4) * d.H + (y0 + rr % 4)) * d.W + x0;
        };
        auto range = [&](int rr) { return z + rr / 4 < d.D && y0 + rr % 4 < d.H ? int(kRange) : 0; };

        __syncthreads();  // this item's tiles are in LDS
        // What the epilogue reads is loaded ahead of the products.
        constexpr bool kReads = kOut == kLoss || kOut == kGate;
        static_assert(!kReads || RZ == 1, "8 rows leave no registers for them");
        uint32_t tg[kOut == kLoss ? NR4 : 1][4];
        v2u zg[kOut == kGate ? NR4 : 1][NCO];
        if (kReads && last && kg == 0) {
#pragma unroll
            for (int rr = 0; rr < NR4; ++rr) {
                if constexpr (kOut == kLoss) {
                    const auto r = buffer_of(ls.target + row0(rr) * ls.K, range(rr));
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const int c = co0 + kq * 4 + k;
                        tg[rr][k] = __builtin_amdgcn_raw_buffer_load_b32(
                            r, xin && c < ls.K ? uint32_t(col * ls.K + c) * 4 : kOutside, 0, 0);
                    }
                } else if constexpr (kOut == kGate) {
#pragma unroll
                    for (int j = 0; j < NCO; ++j)
                        zg[rr][j] = load_vec<kDirect>(ep.gate + row0(rr) * Co + co0, range(rr),
                                                      xin ? uint32_t(col * Co + j * 16 + kq * 4) * 2 : kOutside);
                }
            }
        }
        if (NBUF > 1)
            load_item(item + 1);
        const int boff = NBUF > 1 ? (item & 1) * int(sizeof(Tile) / sizeof(bf)) : 0;
        // 14 tap pairs (27 taps and a zero tap), each a K = 32 product.
        // Each input operand is read at its first use and kept for the later ones.
        if (active) {
            constexpr FirstUse<RZ> first;
            bf8v wv8[kAhead ? 2 : 1][NCO], v[3][RZ + 2][FC_HY], v1[NR4];
            auto read_pair = [&](int pr) {
                const int kd = TapPairs::kind[pr], dz = TapPairs::dz[pr], dy = TapPairs::dy[pr];
#pragma unroll
                for (int jj = 0; jj < NCO; ++jj)
                    wv8[kAhead ? pr & 1 : 0][jj] = *reinterpret_cast<const bf8v *>(wa + boff + (2 * pr * NCO + jj) * 256);
#pragma unroll
                for (int rr = 0; rr < NR4; ++rr) {
                    const int z = rr / 4, y = rr % 4;
                    if (kd == 3)
                        v1[rr] = *reinterpret_cast<const bf8v *>(at[3] + boff + (z * FC_HY + y) * FC_ROW);
                    else if (kd == 4)
                        v1[rr] = *reinterpret_cast<const bf8v *>(at[4 + z] + boff + y * FC_ROW);
                    else if (first.pair[kd][z + dz][y + dy] == pr)
                        v[kd][z + dz][y + dy] =
                            *reinterpret_cast<const bf8v *>(at[kd] + boff + ((z + dz) * FC_HY + y + dy) * FC_ROW);
                }
            };
            // With two waves per SIMD the next pair's operands are read while the
            // current pair's products run (the scheduling barriers keep the reads
            // ahead of the products); more waves cover the reads by themselves.
            if (kAhead)
                read_pair(0);
#pragma unroll
            for (int pr = 0; pr < 14; ++pr) {
                const int kd = TapPairs::kind[pr], dz = TapPairs::dz[pr], dy = TapPairs::dy[pr];
                bf8v bv[NR4];
                if (!kAhead)
                    read_pair(pr);
#pragma unroll
                for (int rr = 0; rr < NR4; ++rr)
                    bv[rr] = kd < 3 ? v[kd][rr / 4 + dz][rr % 4 + dy] : v1[rr];
                if (kAhead) {
                    if (pr + 1 < 14)
                        read_pair(pr + 1);
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int rr = 0; rr < NR4; ++rr)
#pragma unroll
                    for (int jj = 0; jj < NCO; ++jj)
                        acc[rr][jj] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv8[kAhead ? pr & 1 : 0][jj], bv[rr],
                                                                              acc[rr][jj], 0, 0, 0);
                if (kAhead)
                    __builtin_amdgcn_sched_barrier(0);
            }
        }
        if constexpr (NBUF == 1) {
            // The next item's loads are on their way while this brick's results
            // are finished and stored, and are waited for but not the stores.
            if constexpr (kReads)  // the epilogue's operands have arrived: no wait for them after these loads
#pragma unroll
                for (int rr = 0; rr < NR4; ++rr) {
                    if constexpr (kOut == kLoss)
                        asm volatile("" : "+v"(tg[rr][0]), "+v"(tg[rr][1]), "+v"(tg[rr][2]), "+v"(tg[rr][3]));
                    else
                        for (int j = 0; j < NCO; ++j)
                            asm volatile("" : "+v"(zg[rr][j]));
                }
            __syncthreads();  // this item's tiles are no longer read
            load_item(item + 1);
        }
        if (!last) {  // more input channels of this brick to accumulate
            wait_loads();
            continue;
        }
        if constexpr (KS > 1) {
            const int cur = item & 1;
            auto red = [&](int g, int rr, int j) -> f4 & {
                return reinterpret_cast<f4 *>(tiles[g][cur].x)[(rr * NCO + j) * FC_THREADS + tid];
            };
            __syncthreads();  // the round's operands are no longer read
            if (kg > 0)
#pragma unroll
                for (int rr = 0; rr < NR4; ++rr)
#pragma unroll
                    for (int j = 0; j < NCO; ++j)
                        red(kg, rr, j) = acc[rr][j];
            __syncthreads();
            if (kg == 0)
                for (int g = 1; g < KS; ++g)
#pragma unroll
                    for (int rr = 0; rr < NR4; ++rr)
#pragma unroll
                        for (int j = 0; j < NCO; ++j)
                            acc[rr][j] += red(g, rr, j);
        }
        asm volatile("" ::: "memory");  // no store moves ahead of the loads
        if (kg == 0) {
#pragma unroll
            for (int rr = 0; rr < NR4; ++rr) {
                const int rows = range(rr);
                const long long p = row0(rr);
#pragma unroll
                for (int j = 0; j < NCO; ++j) {
                    const int cb = j * 16 + kq * 4;  // from co0: this lane's 4 consecutive output channels
                    const f4 v = acc[rr][j] + bj[j];
                    if constexpr (kOut == kF32 || kOut == kLoss) {
                        float *const o = reinterpret_cast<float *>(out);
                        store_vec<kDirect>(o + p * Co + co0, o ? rows : 0, __builtin_bit_cast(v4u, v),
                                           xin ? uint32_t(col * Co + cb) * 4 : kOutside);
                    }
                    if constexpr (kOut == kLoss) {
                        float gv[4];
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            gv[k] = 0.f;
                            if (xin && rows && co0 + cb + k < ls.K) {
                                const float e = v[k] - __uint_as_float(tg[rr][k]);
                                sq += double(e) * e;
                                gv[k] = 2.f * e * ls.scale;
                            }
                        }
                        store_vec<kDirect>(ls.grad + p * Co + co0, rows,
                                           v2u{uint32_t(f2bf(gv[0])) | (uint32_t(f2bf(gv[1])) << 16),
                                               uint32_t(f2bf(gv[2])) | (uint32_t(f2bf(gv[3])) << 16)},
                                           xin ? uint32_t(col * Co + cb) * 2 : kOutside);
                    }
                    if constexpr (kOut == kBf16 || kOut == kAct || kOut == kSilu || kOut == kGate) {
                        bf o[4] = {f2bf(v[0]), f2bf(v[1]), f2bf(v[2]), f2bf(v[3])};
                        if constexpr (kOut == kAct || kOut == kSilu) {
                            const v2u pa{
                                uint32_t(f2bf(silu_f(bf2f(o[0])))) | (uint32_t(f2bf(silu_f(bf2f(o[1])))) << 16),
                                uint32_t(f2bf(silu_f(bf2f(o[2])))) | (uint32_t(f2bf(silu_f(bf2f(o[3])))) << 16)};
                            store_vec<kDirect>(ep.act + p * Co + co0, rows, pa,
                                               xin ? uint32_t(col * Co + cb) * 2 : kOutside);
                        }
                        if constexpr (kOut == kGate) {
                            const v2u q = zg[rr][j];
                            const bf zz[4] = {bf(q.x & 0xffffu), bf(q.x >> 16), bf(q.y & 0xffffu), bf(q.y >> 16)};
#pragma unroll
                            for (int k = 0; k < 4; ++k)
                                o[k] = f2bf(silu_grad_f(bf2f(o[k]), bf2f(zz[k])));
                        }
                        if constexpr (kOut == kSilu)
                            continue;
                        // a channel tile lies on one side of the split
                        const bool two = ep.split > 0 && co0 + j * 16 >= ep.split;
                        const int cs = two ? Co - ep.split : ep.split > 0 ? ep.split : Co;
                        bf *const t = (two ? ep.out2 - ep.split : reinterpret_cast<bf *>(out)) + co0 + j * 16;
                        store_vec<kDirect>(t + p * cs, rows,
                                           v2u{uint32_t(o[0]) | (uint32_t(o[1]) << 16),
                                               uint32_t(o[2]) | (uint32_t(o[3]) << 16)},
                                           xin ? uint32_t(col * cs + kq * 4) * 2 : kOutside);
                    }
                }
            }
        }
        // All but this brick's stores (every lane's, also those out of range).
        constexpr int kStores = NR4 * NCO * (kOut == kAct || kOut == kLoss ? 2 : 1);
        if constexpr (NBUF == 1 && kDirect)
            wait_loads<kStores>();
        else
            wait_loads();
#pragma unroll
        for (int rr = 0; rr < NR4; ++rr)
#pragma unroll
            for (int j = 0; j < NCO; ++j)
                acc[rr][j] = f4{0.f, 0.f, 0.f, 0.f};
    }
    if constexpr (kOut == kLoss) {
        __shared__ double lred[FC_THREADS / 64];
        for (int o = 32; o > 0; o >>= 1)
            sq += __shfl_xor(sq, o);
        if (lane == 0)
            lred[wv] = sq;
        __syncthreads();
        const int blk = int(blockIdx.x + blockIdx.y * gridDim.x), nblk = int(gridDim.x * gridDim.y);
        if (tid == 0) {
            double t = 0.0;
            for (int k = 0; k < FC_THREADS / 64; ++k)
                t += lred[k];
            ls.partial[blk] = t;
        }
        if (blk == 0)
            for (int i = nblk + tid; i < ls.npartial; i += FC_THREADS)
                ls.partial[i] = 0.0;
    }
}

// W'[ci][26 - tap][co] = W[co][tap][ci]: the data gradient is a forward
// convolution of the output gradient with W'.
__global__ __launch_bounds__(256) void k_conv_flip(const bf *__restrict__ w, bf *__restrict__ wt, int Ci,
                                                   int Co)
{
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long n = (long long)Co * 27 * Ci;
    if (i >= n)
        return;
    const int ci = int(i % Ci), tap = int((i / Ci) % 27), co = int(i / (27LL * Ci));
    wt[((long long)ci * 27 + (26 - tap)) * Co + co] = w[i];
}

// The flips of many layers in one launch: blockIdx.y selects the layer,
// whose weights start at w + off[l] and whose flipped copy at wt + off[l].
constexpr int FLIP_MAX = 32;
struct FlipSet {
    int count;
    long long off[FLIP_MAX];
    int ci[FLIP_MAX], co[FLIP_MAX];
};

__global__ __launch_bounds__(256) void k_conv_flip_many(const bf *__restrict__ w, bf *__restrict__ wt,
                                                        FlipSet fs)
{
    const int l = blockIdx.y;
    const int Ci = fs.ci[l], Co = fs.co[l];
    const long long n = (long long)Co * 27 * Ci;
    const bf *wl = w + fs.off[l];
    bf *tl = wt + fs.off[l];
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x) {
        const int ci = int(i % Ci), tap = int((i / Ci) % 27), co = int(i / (27LL * Ci));
        tl[((long long)ci * 27 + (26 - tap)) * Co + co] = wl[i];
    }
}

// gw[co][tap][ci] += sum_p gout[p][co] in[p + off(tap)][ci], gb[co] += sum_p gout[p][co].
//
// A block owns one (co tile, ci tile) pair (blockIdx.y) and a range of the chunks
// of 16 x 8 x 4 voxels, in the order of columns along z.  Down a column it keeps
// rings of plane groups in LDS, channel-last as they lie in memory: four groups
// of four input planes of 18 x 10 voxels (planes 4 k - 1 .. 4 k + 2: chunk c reads
// group c and the first two planes of c + 1) and three of four gout planes.  While
// it computes on chunk c, what chunks c + 1 and c + 2 need travels from memory
// straight into LDS (buffer loads to LDS; voxels outside the volume are
// out of the buffer's range and arrive as zeros); one barrier per chunk.
// The reduction runs over voxels, so both MFMA operands need several voxels of one
// channel per lane: ds_read_b64_tr_b16 transposes on the way out of LDS (lane
// layout checked on the device: 16 voxels of 16 channels, 512 consecutive bytes
// read at lane * 8, give lane l channel l % 16 of voxels 4 (l / 16) .. + 3).  K = 32
// of v_mfma_f32_16x16x32_bf16 is two rows of 16 voxels, one read each, so any
// tap's operand is two reads at lane * 8 plus a constant, and the inner loop is
// LDS reads and MFMAs only.
// Four teams of three waves take two of the chunk's rows in y each; wave dx of a
// team accumulates the 9 taps of its x offset: it holds the row pairs of gout of
// the four planes in registers and reads the 3 row pairs (Y, Y + 1) of each of 6
// input planes once; a row pair serves every dz it lies at: 36 products for 22
// reads.  Wave 0 also accumulates the bias gradient against ones.  At the end
// the teams' sums meet in LDS and the block adds them to gw / gb atomically,
// each block from another place on.
// Bound by the block's fixed part (launch, first loads, the teams' sums: 10 us)
// and the blocks' atomic adds to the same elements (4 us of 28 at 64^3), then by
// loads and products, which overlap (loads alone 21 us, products alone 24).  Batch
// 4, bricks transposed through registers -> loaded whole into LDS -> streamed down
// columns, us: 64^3 16 -> 16 51.5 -> 31 -> 28, 48 -> 16 86 -> 53 -> 52, 32^3 96 -> 32 49
// -> 35 -> 31, 16^3 160 -> 64 33 -> 30 -> 19, 64 -> 64 19.3 -> 14.6 -> 14.
// Element indices are 32-bit (the host checks B D H W C < 2^31 and the plane
// extents).
constexpr int WB_X = 16, WB_Y = 8, WB_Z = 4, WB_V = WB_X * WB_Y * WB_Z;
constexpr int WB_HX = WB_X + 2, WB_HY = WB_Y + 2;
constexpr int WB_HV = WB_HX * WB_HY * WB_Z;         // 720 voxels of an input group
constexpr int WB_TEAMS = WB_Y / 2, WB_WAVES = 3 * WB_TEAMS;
constexpr int WB_ILOADS = 24;                       // wave loads of 64 16-byte pieces: input group (2 per wave)
constexpr int WB_GLOADS = 2 * WB_V / 64;            // and gout group
constexpr int WB_IITERS = (WB_ILOADS + WB_WAVES - 1) / WB_WAVES;  // per wave
constexpr int WB_GITERS = (WB_GLOADS + WB_WAVES - 1) / WB_WAVES;
static_assert(WB_ILOADS * 64 >= 2 * WB_HV && WB_ILOADS == WB_IITERS * WB_WAVES, "as many for every wave");

// The operand of two rows of 16 voxels: this lane's channel, 4 voxels of each.
__device__ __forceinline__ bf8v read_rows(const bf *row0, const bf *row1)
{
    using L = __attribute__((address_space(3))) s4;
    const s4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((L *)row0);
    const s4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((L *)row1);
    return __builtin_bit_cast(bf8v, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

template <bool kDirect>
__global__ __launch_bounds__(64 * WB_WAVES) __attribute__((amdgpu_waves_per_eu(3))) void
k_conv_wgrad(ConvIn src, const bf *__restrict__ gout, float *__restrict__ gw, float *__restrict__ gb, Dims d,
             int nbx, int nby, int nbz)
{
    constexpr int NSUM = 27 * 256 + 16;
    __shared__ __attribute__((aligned(16))) union {
        bf ring[4 * WB_ILOADS * 512 + 3 * WB_GLOADS * 512];
        float sums[WB_TEAMS * NSUM];
    } lds;
    const int Ci = d.Ci, Co = d.Co;
    const int CIT = Ci / 16;
    const int ct = blockIdx.y / CIT, it = blockIdx.y % CIT;
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
    const int team = wave / 3, dx = wave % 3;            // dx: x offset + 1
    const int lane = threadIdx.x & 63;
    const bool up = it * 16 < src.cu;      // this block's input channels come from src.low
    const bf *const in = up ? src.low : src.in;
    const int cs = up ? src.cu : Ci - src.cu;            // channel stride of `in`
    const int cin = up ? it * 16 : it * 16 - src.cu;     // channel offset in it

    // This lane's pieces: wave w runs wave loads j = w + 12 k; piece i = 64 j + lane
    // is half i % 2 of voxel i / 2 of the group.  Offsets from the voxel before the
    // chunk's first one in x, y and z (input) and from its first voxel (gout), and
    // positions in the group.
    constexpr uint32_t kUnits = load_units(kDirect);
    const BrickGrid grid(nbx, nby, 1);
    const int sh = up ? 1 : 0;  // corners are even: (x0 + hx) >> 1 = x0 / 2 + (hx >> 1)
    const int Hi = d.H >> sh, Wi = d.W >> sh, Di = d.D >> sh;
    uint32_t ioff[WB_IITERS], ipos[WB_IITERS], goff[WB_GITERS], gpos[WB_GITERS];
#pragma unroll
    for (int k = 0; k < WB_IITERS; ++k) {
        const int hv = ((wave + WB_WAVES * k) * 64 + lane) >> 1, hrow = hv / WB_HX;
        const int hx = hv % WB_HX, hy = hrow % WB_HY, hz = hrow / WB_HY;
        ioff[k] = kUnits * (uint32_t((((hz - 1) >> sh) + 1) * Hi + ((hy - 1) >> sh) + 1) * Wi + ((hx - 1) >> sh) + 1) *
                      uint32_t(cs) +
                  kUnits * uint32_t(cin + (lane & 1) * 8);
        ipos[k] = hz < WB_Z ? tile_pos(hx, hy, hz) : 0u;  // the last wave load's tail is never inside
    }
#pragma unroll
    for (int k = 0; k < WB_GITERS; ++k) {
        const int v = ((wave + WB_WAVES * k) * 64 + lane) >> 1;
        goff[k] = kUnits * (uint32_t(((v >> 7) * d.H + ((v >> 4) & 7)) * d.W + (v & 15)) * uint32_t(Co) +
                            uint32_t(ct * 16 + (lane & 1) * 8));
        gpos[k] = tile_pos(v & 15, (v >> 4) & 7, v >> 7);
    }
    int b = 0, x0 = 0, y0 = 0;  // the column
    auto load_input = [&](int k4, bf *to) {  // planes k4 - 1 .. k4 + 2
        const bf *const base =
            in + (((long long)(b * Di + (k4 >> sh) - 1) * Hi + (y0 >> sh) - 1) * Wi + (x0 >> sh) - 1) * cs;
        const TileRange inside(x0 == 0, y0 == 0, k4 == 0, d.W - x0, d.H - y0, d.D - k4);
#pragma unroll
        for (int k = 0; k < WB_IITERS; ++k)
            if (wave + WB_WAVES * k < WB_ILOADS)
                load_to_lds<kDirect>(base, to + (wave + WB_WAVES * k) * 512, lane,
                                     inside.has(ipos[k]) ? ioff[k] : kOutside);
    };
    auto load_gout = [&](int z0, bf *to) {
        const bf *const base = gout + (((long long)(b * d.D + z0) * d.H + y0) * d.W + x0) * Co;
        const TileRange inside(0, 0, 0, d.W - 1 - x0, d.H - 1 - y0, d.D - 1 - z0);
#pragma unroll
        for (int k = 0; k < WB_GITERS; ++k)
            if (wave + WB_WAVES * k < WB_GLOADS)
                load_to_lds<kDirect>(base, to + (wave + WB_WAVES * k) * 512, lane,
                                     inside.has(gpos[k]) ? goff[k] : kOutside);
    };

    f4 acc[9], accb = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 9; ++t)
        acc[t] = f4{0.f, 0.f, 0.f, 0.f};
    const bf8v ones = __builtin_bit_cast(bf8v, make_uint4(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u));
    const bool bias_wave = dx == 0 && gb != nullptr && it == 0;
    const int ip = (2 * team * WB_HX + dx) * 16 + lane * 4, gp = 2 * team * WB_X * 16 + lane * 4;

    // chunks of this block: a contiguous range; ranges of one XCD are neighbours
    const int nchunks = d.B * nbx * nby * nbz, G = int(gridDim.x), bx = int(blockIdx.x);
    const int range = G % 8 == 0 ? bx % 8 * (G / 8) + bx / 8 : bx;
    const int c0 = int((long long)range * nchunks / G), c1 = int((long long)(range + 1) * nchunks / G);
    int g0 = 0, q = 0;  // ring places of the chunk's input group and gout group
    auto in_at = [&](int k) { return ((g0 + k) & 3) * (WB_ILOADS * 512); };
    auto go_at = [&](int k) { return 4 * WB_ILOADS * 512 + (q + k < 3 ? q + k : q + k - 3) * (WB_GLOADS * 512); };
    auto load_set = [&](bf *to, int z0, int k) {  // what the k-th chunk from the one at z0 needs anew
        load_input(z0 + (k + 1) * WB_Z, to + in_at(k + 1));
        load_gout(z0 + k * WB_Z, to + go_at(k));
    };
    // Between two barriers: the request for what a later chunk needs, and the products
    // of one whose groups lie in LDS.  The one writes no place of the ring that the
    // other reads, and nothing else is written meanwhile, which restrict tells the
    // compiler: without it, it waits for everything on its way before the first
    // transposing read.  What the next chunk reads is requested, waited for and
    // separated by a barrier outside of both.
    auto request = [&](bf *__restrict__ arrive, int z0) { load_set(arrive, z0, 2); };
    auto products = [&](const bf *__restrict__ ring) {
        const bf *const gq = ring + go_at(0) + gp, *const in0 = ring + in_at(0) + ip, *const in1 = ring + in_at(1) + ip;
        bf8v a[WB_Z];  // the team's two rows of gout plane z
#pragma unroll
        for (int Z = 0; Z < WB_Z + 2; ++Z) {
            if (Z < WB_Z) {
                const bf *const row = gq + Z * WB_Y * WB_X * 16;
                a[Z] = read_rows(row, row + WB_X * 16);
                if (bias_wave)
                    accb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[Z], ones, accb, 0, 0, 0);
            }
            const bf *const plane = (Z < WB_Z ? in0 : in1) + Z % WB_Z * WB_HY * WB_HX * 16;
#pragma unroll
            for (int Y = 0; Y < 3; ++Y) {  // dy + 1
                const bf *const row = plane + Y * WB_HX * 16;
                const bf8v v = read_rows(row, row + WB_HX * 16);
#pragma unroll
                for (int kz = 0; kz < 3; ++kz)  // dz + 1
                    if (Z - kz >= 0 && Z - kz < WB_Z)
                        acc[kz * 3 + Y] =
                            __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[Z - kz], v, acc[kz * 3 + Y], 0, 0, 0);
            }
        }
    };
    int none = 0;  // not known to the compiler, which would pass a known address by itself and lose restrict
    asm volatile("" : "+s"(none));
    for (int c = c0; c < c1; ++c) {
        const int colm = c / nbz, cz = c - colm * nbz, z0 = cz * WB_Z;
        const int rest = min(c1 - c, nbz - cz);  // chunks left of the range in this column
        if (c == c0 || cz == 0) {                // a new column
            int zero;
            grid.at(colm, WB_X, WB_Y, 1, b, x0, y0, zero);
            lds_barrier();  // the previous chunk's reads are done
            load_input(z0, lds.ring + in_at(0));
            load_set(lds.ring, z0, 0);
            if (rest > 1)
                load_set(lds.ring, z0, 1);
        }
        if (kDirect && rest > 1) {  // all but the next chunk's
            if (wave < WB_GLOADS - WB_WAVES)
                wait_loads<WB_IITERS + 2>();
            else
                wait_loads<WB_IITERS + 1>();
        } else {
            wait_loads();
        }
        lds_barrier();
        if (rest > 2)
            request(lds.ring + none, z0);
        if (y0 + 2 * team < d.H)  // else both rows lie outside the volume
            products(lds.ring + none);
        g0 = (g0 + 1) & 3;
        q = q == 2 ? 0 : q + 1;
    }
    // The teams' sums in LDS, each [tap][co][ci] and then the bias; every thread
    // adds its share of their total to the global gradient, blocks starting at
    // different places (from the same one they queue at the same addresses).
    float *const red = lds.sums;
    const int col = lane & 15, kq = lane >> 4;
    __syncthreads();
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r)  // D[4 kq + r][col] = sum of co 4 kq + r, ci col
            red[team * NSUM + (3 * t + dx) * 256 + (kq * 4 + r) * 16 + col] = acc[t][r];
    if (dx == 0 && col == 0)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            red[team * NSUM + 27 * 256 + kq * 4 + r] = accb[r];
    __syncthreads();
    auto total = [&](int e) {
        float v = red[e];
        for (int q = 1; q < WB_TEAMS; ++q)
            v += red[q * NSUM + e];
        return v;
    };
    const int rot = int(blockIdx.x) * 7 % 108 * 64;
    for (int k = threadIdx.x; k < 27 * 256; k += 64 * WB_WAVES) {
        int e = k + rot;
        if (e >= 27 * 256)
            e -= 27 * 256;
        const int tap = e >> 8, co = ct * 16 + ((e >> 4) & 15), ci = it * 16 + (e & 15);
        atomicAdd(&gw[(co * 27 + tap) * Ci + ci], total(e));
    }
    if (gb != nullptr && it == 0 && threadIdx.x < 16)
        atomicAdd(&gb[ct * 16 + threadIdx.x], total(27 * 256 + threadIdx.x));
}

// ------------------------------------------------------------ elementwise
// SiLU a = z sigma(z); backward dz = da sigma(z) (1 + z (1 - sigma(z))).
__global__ __launch_bounds__(256) void k_silu_fwd(const bf *__restrict__ z, bf *__restrict__ a, long long n)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x)
        a[i] = f2bf(silu_f(bf2f(z[i])));
}

__global__ __launch_bounds__(256) void k_silu_bwd(const bf *__restrict__ z, const bf *__restrict__ ga,
                                                  bf *__restrict__ gz, long long n)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x)
        gz[i] = f2bf(silu_grad_f(bf2f(ga[i]), bf2f(z[i])));
}

// The vector kernels below move 8 channels (16 bytes) per thread; every
// channel count is a multiple of 16, so a vector never straddles a voxel or
// a concatenation boundary.  Index arithmetic is 32-bit (the launchers check
// the element counts).
__device__ __forceinline__ void unpack8(const uint4 &v, float f[8])
{
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        f[2 * k] = __uint_as_float(w[k] << 16);
        f[2 * k + 1] = __uint_as_float(w[k] & 0xffff0000u);
    }
}
__device__ __forceinline__ uint4 pack8(const float f[8])
{
    uint32_t w[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
        w[k] = uint32_t(f2bf(f[2 * k])) | (uint32_t(f2bf(f[2 * k + 1])) << 16);
    return make_uint4(w[0], w[1], w[2], w[3]);
}

// cat[p] = [up2(h)[p] (Ch channels) | skip[p] (Cs)] on the fine grid
// (2D x 2H x 2W; h on D x H x W): nearest upsampling and concatenation in
// one pass.
__global__ __launch_bounds__(256) void k_upcat(const uint4 *__restrict__ h, const uint4 *__restrict__ skip,
                                               uint4 *__restrict__ cat, int B, int D, int H, int W, int Ch8,
                                               int Cs8)
{
    const int C8 = Ch8 + Cs8, Wo = 2 * W, Ho = 2 * H, Do = 2 * D;
    const uint32_t n = uint32_t(B) * Do * Ho * Wo * C8;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const uint32_t c = i % C8, p = i / C8;
        if (int(c) < Ch8) {
            uint32_t r = p;
            const uint32_t x = r % Wo; r /= Wo;
            const uint32_t y = r % Ho; r /= Ho;
            const uint32_t z = r % Do;
            const uint32_t b = r / Do;
            cat[i] = h[(((b * D + z / 2) * H + y / 2) * W + x / 2) * Ch8 + c];
        } else {
            cat[i] = skip[p * Cs8 + (c - Ch8)];
        }
    }
}

// Gradient through 2x2x2 average pooling, plus an optional second gradient
// of the same tensor (add, the skip connection's), times the optional SiLU
// derivative at z (gate): gin = silu'(z) * (bf16(gout[parent] / 8) + add),
// rounded to BF16 after each step as the separate kernels round.
__global__ __launch_bounds__(256) void k_pool2_bwd_gate(const uint4 *__restrict__ gout,
                                                        const uint4 *__restrict__ add,
                                                        const uint4 *__restrict__ gate,
                                                        uint4 *__restrict__ gin, int B, int D, int H, int W,
                                                        int C8)
{
    const int Do = D / 2, Ho = H / 2, Wo = W / 2;
    const uint32_t n = uint32_t(B) * D * H * W * C8;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        uint32_t r = i;
        const uint32_t c = r % C8; r /= C8;
        const uint32_t x = r % W; r /= W;
        const uint32_t y = r % H; r /= H;
        const uint32_t z = r % D;
        const uint32_t b = r / D;
        float g[8], t[8];
        unpack8(gout[(((b * Do + z / 2) * Ho + y / 2) * Wo + x / 2) * C8 + c], g);
#pragma unroll
        for (int k = 0; k < 8; ++k)
            g[k] = bf2f(f2bf(0.125f * g[k]));
        if (add) {
            unpack8(add[i], t);
#pragma unroll
            for (int k = 0; k < 8; ++k)
                g[k] = bf2f(f2bf(g[k] + t[k]));
        }
        if (gate) {
            unpack8(gate[i], t);
#pragma unroll
            for (int k = 0; k < 8; ++k)
                g[k] = silu_grad_f(g[k], t[k]);
        }
        gin[i] = pack8(g);
    }
}

// Gradient through nearest x2 upsampling (the sum over the 8 copies), times
// the optional SiLU derivative at z (gate), BF16 after each step.
__global__ __launch_bounds__(256) void k_up2_bwd_gate(const uint4 *__restrict__ gout,
                                                      const uint4 *__restrict__ gate,
                                                      uint4 *__restrict__ gin, int B, int D, int H, int W,
                                                      int C8)
{
    const int Do = 2 * D, Ho = 2 * H, Wo = 2 * W;
    const uint32_t n = uint32_t(B) * D * H * W * C8;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        uint32_t r = i;
        const uint32_t c = r % C8; r /= C8;
        const uint32_t x = r % W; r /= W;
        const uint32_t y = r % H; r /= H;
        const uint32_t z = r % D;
        const uint32_t b = r / D;
        float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, t[8];
        for (int k = 0; k < 8; ++k) {
            const uint32_t xo = 2 * x + (k & 1), yo = 2 * y + ((k >> 1) & 1), zo = 2 * z + (k >> 2);
            unpack8(gout[(((b * Do + zo) * Ho + yo) * Wo + xo) * C8 + c], t);
#pragma unroll
            for (int q = 0; q < 8; ++q)
                s[q] += t[q];
        }
        if (gate) {
#pragma unroll
            for (int q = 0; q < 8; ++q)
                s[q] = bf2f(f2bf(s[q]));
            unpack8(gate[i], t);
#pragma unroll
            for (int q = 0; q < 8; ++q)
                s[q] = silu_grad_f(s[q], t[q]);
        }
        gin[i] = pack8(s);
    }
}

// 2x2x2 average pooling (even D, H, W) and its gradient.
__global__ __launch_bounds__(256) void k_pool2_fwd(const bf *__restrict__ in, bf *__restrict__ out, int B,
                                                   int D, int H, int W, int C)
{
    const int Do = D / 2, Ho = H / 2, Wo = W / 2;
    const long long n = (long long)B * Do * Ho * Wo * C;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x) {
        long long r = i;
        const int c = int(r % C); r /= C;
        const int x = int(r % Wo); r /= Wo;
        const int y = int(r % Ho); r /= Ho;
        const int z = int(r % Do);
        const int b = int(r / Do);
        float s = 0.f;
        for (int k = 0; k < 8; ++k) {
            const int xi = 2 * x + (k & 1), yi = 2 * y + ((k >> 1) & 1), zi = 2 * z + (k >> 2);
            s += bf2f(in[((((long long)b * D + zi) * H + yi) * W + xi) * C + c]);
        }
        out[i] = f2bf(0.125f * s);
    }
}

__global__ __launch_bounds__(256) void k_pool2_bwd(const bf *__restrict__ gout, bf *__restrict__ gin, int B,
                                                   int D, int H, int W, int C)
{
    const long long n = (long long)B * D * H * W * C;
    const int Do = D / 2, Ho = H / 2, Wo = W / 2;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x) {
        long long r = i;
        const int c = int(r % C); r /= C;
        const int x = int(r % W); r /= W;
        const int y = int(r % H); r /= H;
        const int z = int(r % D);
        const int b = int(r / D);
        gin[i] = f2bf(0.125f * bf2f(gout[((((long long)b * Do + z / 2) * Ho + y / 2) * Wo + x / 2) * C + c]));
    }
}

// 2x2x2 average pooling, 8 channels (16 bytes) per thread; the same sums in
// the same order as k_pool2_fwd.
__global__ __launch_bounds__(256) void k_pool2_fwd8(const uint4 *__restrict__ in, uint4 *__restrict__ out,
                                                    int B, int D, int H, int W, int C8)
{
    const int Do = D / 2, Ho = H / 2, Wo = W / 2;
    const uint32_t n = uint32_t(B) * Do * Ho * Wo * C8;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        uint32_t r = i;
        const uint32_t c = r % C8; r /= C8;
        const uint32_t x = r % Wo; r /= Wo;
        const uint32_t y = r % Ho; r /= Ho;
        const uint32_t z = r % Do;
        const uint32_t b = r / Do;
        float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, t[8];
        for (int k = 0; k < 8; ++k) {
            const uint32_t xi = 2 * x + (k & 1), yi = 2 * y + ((k >> 1) & 1), zi = 2 * z + (k >> 2);
            unpack8(in[(((b * D + zi) * H + yi) * W + xi) * C8 + c], t);
#pragma unroll
            for (int q = 0; q < 8; ++q)
                s[q] += t[q];
        }
#pragma unroll
        for (int q = 0; q < 8; ++q)
            s[q] *= 0.125f;
        out[i] = pack8(s);
    }
}

// Nearest-neighbour x2 upsampling (out is 2D x 2H x 2W) and its gradient.
__global__ __launch_bounds__(256) void k_up2_fwd(const bf *__restrict__ in, bf *__restrict__ out, int B,
                                                 int D, int H, int W, int C)
{
    const int Do = 2 * D, Ho = 2 * H, Wo = 2 * W;
    const long long n = (long long)B * Do * Ho * Wo * C;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x) {
        long long r = i;
        const int c = int(r % C); r /= C;
        const int x = int(r % Wo); r /= Wo;
        const int y = int(r % Ho); r /= Ho;
        const int z = int(r % Do);
        const int b = int(r / Do);
        out[i] = in[((((long long)b * D + z / 2) * H + y / 2) * W + x / 2) * C + c];
    }
}

__global__ __launch_bounds__(256) void k_up2_bwd(const bf *__restrict__ gout, bf *__restrict__ gin, int B,
                                                 int D, int H, int W, int C)
{
    const long long n = (long long)B * D * H * W * C;
    const int Do = 2 * D, Ho = 2 * H, Wo = 2 * W;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x) {
        long long r = i;
        const int c = int(r % C); r /= C;
        const int x = int(r % W); r /= W;
        const int y = int(r % H); r /= H;
        const int z = int(r % D);
        const int b = int(r / D);
        float s = 0.f;
        for (int k = 0; k < 8; ++k) {
            const int xo = 2 * x + (k & 1), yo = 2 * y + ((k >> 1) & 1), zo = 2 * z + (k >> 2);
            s += bf2f(gout[((((long long)b * Do + zo) * Ho + yo) * Wo + xo) * C + c]);
        }
        gin[i] = f2bf(s);
    }
}

// Channel concatenation out[p] = [a[p] (Ca) | b[p] (Cb)] and its split.
__global__ __launch_bounds__(256) void k_concat(const bf *__restrict__ a, const bf *__restrict__ b,
                                                bf *__restrict__ out, long long nv, int Ca, int Cb)
{
    const int C = Ca + Cb;
    const long long n = nv * C;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x) {
        const long long p = i / C;
        const int c = int(i % C);
        out[i] = c < Ca ? a[p * Ca + c] : b[p * Cb + (c - Ca)];
    }
}

__global__ __launch_bounds__(256) void k_split(const bf *__restrict__ g, bf *__restrict__ ga,
                                               bf *__restrict__ gb, long long nv, int Ca, int Cb)
{
    const int C = Ca + Cb;
    const long long n = nv * C;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x) {
        const long long p = i / C;
        const int c = int(i % C);
        if (c < Ca)
            ga[p * Ca + c] = g[i];
        else
            gb[p * Cb + (c - Ca)] = g[i];
    }
}

// Mean squared error over the first K channels of pred [nv][C] (FP32)
// against target [nv][K] (FP32); gradient written as BF16 [nv][C] (zero in
// channels >= K); per-block partial sums of squared errors in partial[].
__global__ __launch_bounds__(256) void k_mse(const float *__restrict__ pred, const float *__restrict__ target,
                                             bf *__restrict__ grad, double *__restrict__ partial,
                                             long long nv, int C, int K, float scale)
{
    __shared__ double red[256];
    double s = 0.0;
    const long long n = nv * C;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x) {
        const long long p = i / C;
        const int c = int(i % C);
        float g = 0.f;
        if (c < K) {
            const float e = pred[i] - target[p * K + c];
            s += double(e) * e;
            g = 2.f * e * scale;
        }
        grad[i] = f2bf(g);
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int o = blockDim.x / 2; o > 0; o >>= 1) {
        if (threadIdx.x < o)
            red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0)
        partial[blockIdx.x] = red[0];
}

// The same loss and gradient, one voxel per thread for C % 8 == 0 and
// K <= 8: only the K predicted channels are read, and the gradient row is
// written 8 channels (16 bytes) at a time.
__global__ __launch_bounds__(256) void k_mse_v(const float *__restrict__ pred, const float *__restrict__ target,
                                               uint4 *__restrict__ grad, double *__restrict__ partial,
                                               long long nv, int C, int K, float scale)
{
    __shared__ double red[256];
    double s = 0.0;
    const int C8 = C / 8;
    for (long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x; p < nv;
         p += (long long)gridDim.x * blockDim.x) {
        float g[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        for (int c = 0; c < K; ++c) {
            const float e = pred[p * C + c] - target[p * K + c];
            s += double(e) * e;
            g[c] = 2.f * e * scale;
        }
        grad[p * C8] = pack8(g);
        const uint4 zero = make_uint4(0, 0, 0, 0);
        for (int c8 = 1; c8 < C8; ++c8)
            grad[p * C8 + c8] = zero;
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int o = blockDim.x / 2; o > 0; o >>= 1) {
        if (threadIdx.x < o)
            red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0)
        partial[blockIdx.x] = red[0];
}

// Adam with decoupled weight decay on FP32 master weights; refreshes the
// BF16 copy (nullable) and clears the gradient.
// With wt (not null), also the flipped BF16 copies of the layers in fs
// (offsets ascending), as k_conv_flip_many of wb would write them.
__global__ __launch_bounds__(256) void k_adam(float *__restrict__ w, float *__restrict__ g,
                                              float *__restrict__ m, float *__restrict__ v,
                                              bf *__restrict__ wb, long long n, float lr, float b1,
                                              float b2, float eps, float c1, float c2, float wd,
                                              bf *__restrict__ wt, FlipSet fs)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x) {
        const float gi = g[i];
        const float mi = b1 * m[i] + (1.f - b1) * gi;
        const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
        m[i] = mi;
        v[i] = vi;
        const float wi = w[i] - lr * ((mi * c1) / (sqrtf(vi * c2) + eps) + wd * w[i]);
        w[i] = wi;
        if (wb)
            wb[i] = f2bf(wi);
        g[i] = 0.f;
        if (wt) {
            int l = 0;
            while (l + 1 < fs.count && fs.off[l + 1] <= i)
                ++l;
            const long long local = i - fs.off[l];
            const int Ci = fs.ci[l], Co = fs.co[l];
            if (local >= 0 && local < (long long)Co * 27 * Ci) {
                const int li = int(local);
                const int ci = li % Ci, tap = (li / Ci) % 27, co = li / (27 * Ci);
                wt[fs.off[l] + ((long long)ci * 27 + (26 - tap)) * Co + co] = f2bf(wi);
            }
        }
    }
}

__global__ __launch_bounds__(256) void k_f32_to_bf16(const float *__restrict__ a, bf *__restrict__ b, long long n)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x)
        b[i] = f2bf(a[i]);
}

// Network input on an m^3 node-centred grid, 16 channels per voxel:
// normalised log10 Ra, one-hot wall type (3), node coordinates in [-1, 1]
// (3), zeros.  cond[b] = {log-Ra feature, wall type}.  Block r writes the
// row r = (b m + z) m + y of voxels, thread t the 16-byte pieces t, t + 128,
// ... of the row (piece 2x: voxel x's first 8 channels, 2x + 1: its zeros),
// so each store instruction covers a contiguous run; the row's indices and
// coordinates are computed once per block.
__global__ __launch_bounds__(128) void k_make_input(const float *__restrict__ cond, bf *__restrict__ out, int m)
{
    const int r = int(blockIdx.x);
    const int y = r % m, z = (r / m) % m, b = r / (m * m);
    const float lra = cond[2 * b], wt = cond[2 * b + 1];
    float ch[8] = {lra, wt == 1.f ? 1.f : 0.f, wt == 2.f ? 1.f : 0.f, wt == 3.f ? 1.f : 0.f, 0.f,
                   (2.f * y + 1.f) / m - 1.f, (2.f * z + 1.f) / m - 1.f, 0.f};
    uint4 *o = reinterpret_cast<uint4 *>(out + size_t(r) * m * 16);  // 32 bytes per voxel
    for (int p = int(threadIdx.x); p < 2 * m; p += int(blockDim.x)) {
        uint4 v = make_uint4(0, 0, 0, 0);
        if ((p & 1) == 0) {
            ch[4] = (2.f * (p >> 1) + 1.f) / m - 1.f;
            v = pack8(ch);
        }
        o[p] = v;
    }
}

// Channel-first [B][K][V] <-> channel-last [B][V][C] (first K of C channels), FP32.
// (channel-last value) = (channel-first value) * scale[k] (scale may be null).
__global__ __launch_bounds__(256) void k_cf_to_cl(const float *__restrict__ a, float *__restrict__ b, int B,
                                                  long long V, int K, int C, const float *__restrict__ scale)
{
    const long long n = (long long)B * V * C;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x) {
        const int c = int(i % C);
        const long long v = (i / C) % V, bb = i / (C * V);
        b[i] = c < K ? a[(bb * K + c) * V + v] * (scale ? scale[c] : 1.f) : 0.f;
    }
}

__global__ __launch_bounds__(256) void k_cl_to_cf(const float *__restrict__ a, float *__restrict__ b, int B,
                                                  long long V, int K, int C, const float *__restrict__ scale)
{
    const long long n = (long long)B * K * V;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x) {
        const long long v = i % V;
        const int k = int((i / V) % K);
        const long long bb = i / (V * K);
        b[i] = a[(bb * V + v) * C + k] * (scale ? scale[k] : 1.f);
    }
}

// Channel-first [B][K][m^3] -> channel-last [B][m^3][C] (first K of C
// channels) on a cubic grid, with axis flips and per-channel signs: output
// voxel (x, y, z) takes input voxel (x', y', z'), x' = m - 1 - x if flip & 1
// (y: & 2, z: & 4), else x; channel k times sign[k] * scale[k].
struct ChannelSigns {
    float s[8];
};
__global__ __launch_bounds__(256) void k_cf_to_cl_flip(const float *__restrict__ a, float *__restrict__ b,
                                                       int B, int m, int K, int C, int flip, ChannelSigns sg,
                                                       const float *__restrict__ scale)
{
    const long long V = (long long)m * m * m;
    const long long n = (long long)B * V * C;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x) {
        const int c = int(i % C);
        const long long v = (i / C) % V, bb = i / (C * V);
        if (c >= K) {
            b[i] = 0.f;
            continue;
        }
        int x = int(v % m), y = int((v / m) % m), z = int(v / ((long long)m * m));
        if (flip & 1) x = m - 1 - x;
        if (flip & 2) y = m - 1 - y;
        if (flip & 4) z = m - 1 - z;
        const long long vs = ((long long)z * m + y) * m + x;
        b[i] = a[(bb * K + c) * V + vs] * sg.s[c] * (scale ? scale[c] : 1.f);
    }
}

// out = a + b (BF16, computed in FP32).
__global__ __launch_bounds__(256) void k_add(const bf *__restrict__ a, const bf *__restrict__ b,
                                             bf *__restrict__ out, long long n)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x)
        out[i] = f2bf(bf2f(a[i]) + bf2f(b[i]));
}

unsigned blocks_for(long long n)
{
    long long b = (n + 255) / 256;
    return unsigned(b < 8192 ? (b < 1 ? 1 : b) : 8192);
}

hipStream_t S(void *s) { return reinterpret_cast<hipStream_t>(s); }

lbmx_status check_dims(int B, int D, int H, int W)
{
    if (B < 1 || D < 1 || H < 1 || W < 1)
        return fail(LBMX_EINVAL, "tensor extents must be positive");
    return LBMX_OK;
}

// Whether every pointer is a multiple of 16 bytes (null counts).
template <class... P>
bool aligned16(const P *...p)
{
    return ((reinterpret_cast<uintptr_t>(p) | ... | 0) & 15) == 0;
}

// Compute units of the current device.
int compute_units()
{
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
        cus = 256;
    return cus;
}

template <int NCO, int RZ, FcOut kOut, int KS, bool kDirect>
void launch_fwd_as(ConvIn src, const bf *w, const float *bias, void *out, Dims d, int cus, hipStream_t s, Epilogue ep,
                   LossEp ls = LossEp{})
{
    const int nbx = (d.W + FC_X - 1) / FC_X, nby = (d.H + FC_Y - 1) / FC_Y, nbz = (d.D + 4 * RZ - 1) / (4 * RZ);
    const unsigned bricks = unsigned(d.B * nbx * nby * nbz);
    const unsigned groups = unsigned(d.Co / 16 / NCO);
    // One wave of resident blocks, each walking several bricks so that the
    // next brick's loads overlap the current one's products (measured 2-3 %
    // faster than one brick per block on the 64^3 layers); their number is
    // kept a multiple of 8 for the XCD-aware brick order.  With fewer bricks than
    // that, one each (8 blocks for 12 bricks, a batch of 3 at 8^3: 96 -> 96 16.0
    // us, 12 blocks 9.7).
    static const int per_cu = [] {
        int nb = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_conv_fwd<NCO, RZ, kOut, KS, kDirect>,
                                                         FC_THREADS * KS, 0) != hipSuccess)
            nb = 1;
        return nb < 1 ? 1 : nb;
    }();
    const unsigned resident = unsigned(per_cu) * unsigned(cus) / groups;
    unsigned grid = std::max(1u, std::min(bricks, resident));
    if (kOut == kLoss)  // one partial sum per block
        grid = std::max(1u, std::min(grid, unsigned(ls.npartial) / groups));
    if (grid < bricks && grid >= 8)
        grid -= grid % 8;
    hipLaunchKernelGGL((k_conv_fwd<NCO, RZ, kOut, KS, kDirect>), dim3(grid, groups), dim3(FC_THREADS * KS), 0, s, src, w,
                       bias, out, d, nbx, nby, nbz, ep, ls);
}

template <int NCO, int RZ, int KS = 1, bool kDirect = true>
void launch_fwd(ConvIn src, const bf *w, const float *bias, void *out, int out_f32, Dims d, int cus, hipStream_t s,
                Epilogue ep)
{
    const auto run = out_f32   ? launch_fwd_as<NCO, RZ, kF32, KS, kDirect>
                     : ep.act  ? out ? launch_fwd_as<NCO, RZ, kAct, KS, kDirect>
                                     : launch_fwd_as<NCO, RZ, kSilu, KS, kDirect>
                     : ep.gate ? launch_fwd_as<NCO, 1, kGate, KS, kDirect>  // 8 rows leave no registers for the gate
                               : launch_fwd_as<NCO, RZ, kBf16, KS, kDirect>;
    run(src, w, bias, out, d, cus, s, ep, LossEp{});
}

// Rejects planes whose brick-relative element offsets (a few planes of
// H W voxels of C channels, computed once per thread in 32 bits) overflow.
lbmx_status check_plane(int32_t H, int32_t W, int32_t C, const char *what)
{
    if (6 * ((long long)H + 1) * ((long long)W + 2) * C >= (1LL << 31))
        return fail(LBMX_EINVAL, "%s: H W planes too large for 32-bit brick offsets (need "
                                 "6 (H + 1) (W + 2) C < 2^31)", what);
    return LBMX_OK;
}

// Rejects an upsample-and-concatenate input whose low part is malformed.
lbmx_status check_upcat(const ConvIn &src, int32_t D, int32_t H, int32_t W, int32_t Ci, const char *what)
{
    if (!src.low)
        return LBMX_OK;
    if (src.cu < 16 || src.cu % 16 || src.cu >= Ci)
        return fail(LBMX_EINVAL, "%s: need upsampled channels a multiple of 16 below the total", what);
    if (D % 2 || H % 2 || W % 2)
        return fail(LBMX_EINVAL, "%s: upsampling needs even D, H, W", what);
    return LBMX_OK;
}

// out may be null where act_only allows it: the activation alone is written.
lbmx_status conv_fwd(ConvIn src, const void *w, const float *bias, void *out, int32_t out_f32,
                     int32_t B, int32_t D, int32_t H, int32_t W, int32_t Ci, int32_t Co, void *stream,
                     Epilogue ep, bool act_only = false)
{
    lbmx_status st = check_dims(B, D, H, W);
    if (st != LBMX_OK)
        return st;
    if (!src.in || !w || (!out && !(act_only && ep.act)))
        return fail(LBMX_EINVAL, "conv3d: NULL tensor");
    if (Ci < 16 || Ci % 16 || Ci > 1024 || Co < 16 || Co % 16 || Co > 1024)
        return fail(LBMX_EINVAL, "conv3d: need Ci, Co multiples of 16 in [16, 1024]");
    if ((long long)B * D * H * W >= (1LL << 31))
        return fail(LBMX_EINVAL, "conv3d: %lld voxels exceed 32-bit voxel indices",
                    (long long)B * D * H * W);
    if (out_f32 && (ep.act || ep.gate || ep.out2))
        return fail(LBMX_EINVAL, "conv3d: epilogue options need a BF16 output");
    if (ep.out2 && (ep.split <= 0 || ep.split >= Co || ep.split % 16 || ep.act || ep.gate))
        return fail(LBMX_EINVAL, "conv3d: split must be a multiple of 16 in (0, Co), without act or gate");
    if (ep.act && ep.gate)
        return fail(LBMX_EINVAL, "conv3d: act and gate exclude each other");
    if (!ep.out2)
        ep.split = 0;
    if ((st = check_upcat(src, D, H, W, Ci, "conv3d")) != LBMX_OK ||
        (st = check_plane(H, W, Ci, "conv3d")) != LBMX_OK)
        return st;
    const Dims d{B, D, H, W, Ci, Co};
    const bf *wb = reinterpret_cast<const bf *>(w);
    hipStream_t s = S(stream);
    // Two or three output channel tiles per block (the input tile is staged
    // once for them) where that leaves two blocks per CU (on smaller grids more
    // blocks hide more latency): batch 4, 16 -> 48 at 64^3 54 us with one, 47 with
    // three.  Bricks of 8 planes with one tile from eight blocks per CU on and as
    // far as 32-bit offsets over their halo go: 16 -> 16 at 64^3 29.1 -> 26.8 us,
    // 48 -> 16 59 -> 52, but at batch 1 17.6 -> 19.9, and with a gate, whose loads no
    // register is free for during the products, 29.7 -> 31.3 (they fill the 168
    // registers of three waves per SIMD and spill 7 or 8 of them; with two tiles the
    // spills cost what the bricks gain).  Two groups per block that split the rounds when
    // one tile per block leaves at most one block per CU.  Operands that are not
    // 16-byte aligned take the smallest tile with the same split.
    const long long bricks =
        (long long)B * ((W + FC_X - 1) / FC_X) * ((H + FC_Y - 1) / FC_Y) * ((D + 3) / 4);
    const int tiles = Co / 16, cus = compute_units();
    const bool far = 2LL * (4 * 2 + 3) * (H + 1) * (W + 2) * Ci >= (long long)kRange;
    const bool two = tiles % 2 == 0 && bricks * (tiles / 2) >= 2 * cus;
    const bool split = !two && Ci >= 32 && bricks * tiles <= cus;
    if (!aligned16(src.in, src.low, wb, reinterpret_cast<bf *>(out), ep.act, ep.gate, ep.out2)) {
        if (split)
            launch_fwd<1, 1, 2, false>(src, wb, bias, out, out_f32, d, cus, s, ep);
        else
            launch_fwd<1, 1, 1, false>(src, wb, bias, out, out_f32, d, cus, s, ep);
    } else if (two)
        launch_fwd<2, 1>(src, wb, bias, out, out_f32, d, cus, s, ep);
    else if (tiles % 3 == 0 && bricks * (tiles / 3) >= 2 * cus)
        launch_fwd<3, 1>(src, wb, bias, out, out_f32, d, cus, s, ep);
    else if (split)
        launch_fwd<1, 1, 2>(src, wb, bias, out, out_f32, d, cus, s, ep);
    else if (!far && bricks * tiles >= 8 * cus)
        launch_fwd<1, 2>(src, wb, bias, out, out_f32, d, cus, s, ep);
    else
        launch_fwd<1, 1>(src, wb, bias, out, out_f32, d, cus, s, ep);
    HIP_TRY(hipGetLastError());
    return LBMX_OK;
}

// The U-Net's inference: every launch in order, activations one after another
// in the workspace (base null: only its size is counted).
struct UnetPlan {
    const int32_t *levels;
    int count, B, m;
    void *stream;
    char *base;
    size_t used = 0;

    bf *take(int r, int c)
    {
        char *const p = base ? base + used : nullptr;
        used += (size_t(B) * r * r * r * c * sizeof(bf) + 255) / 256 * 256;
        return reinterpret_cast<bf *>(p);
    }
    lbmx_status run(const float *cond, const void *const *w, const float *const *b, float *pred)
    {
        int q = 0, r = m;
        lbmx_status st = LBMX_OK;
        auto layer = [&](ConvIn src, int ci, int co, lbmx_status *s) {
            bf *const a = take(r, co);
            if (base && *s == LBMX_OK)
                *s = conv_fwd(src, w[q], b[q], nullptr, 0, B, r, r, r, ci, co, stream,
                              Epilogue{a, nullptr, nullptr, 0}, true);
            ++q;
            return a;
        };
        bf *h = take(r, 16);
        if (base)
            st = lbmx_nn_make_input(cond, h, B, m, stream);
        int ch = 16;
        bf *skip[8];
        for (int l = 0; l < count; ++l) {
            const int c = levels[l];
            h = layer(ConvIn{h, nullptr, 0}, ch, c, &st);
            h = layer(ConvIn{h, nullptr, 0}, c, c, &st);
            ch = c;
            if (l + 1 < count) {
                skip[l] = h;
                bf *const p = take(r / 2, c);
                if (base && st == LBMX_OK)
                    st = lbmx_nn_pool2(h, p, B, r, r, r, c, 0, stream);
                h = p;
                r /= 2;
            }
        }
        for (int l = count - 2; l >= 0; --l) {
            const int c = levels[l];
            r *= 2;
            h = layer(ConvIn{skip[l], h, ch}, ch + c, c, &st);
            h = layer(ConvIn{h, nullptr, 0}, c, c, &st);
            ch = c;
        }
        if (base && st == LBMX_OK)
            st = lbmx_nn_conv3d_fwd(h, w[q], b[q], pred, 1, B, m, m, m, ch, 16, stream);
        return st;
    }
};

lbmx_status check_unet(const int32_t *levels, int32_t count, int32_t B, int32_t m)
{
    if (!levels || count < 1 || count > 8 || B < 1 || m < 1 || m > 4096)
        return fail(LBMX_EINVAL, "unet: need 1 to 8 levels, B >= 1 and 1 <= m <= 4096");
    for (int l = 0; l < count; ++l)
        if (levels[l] < 16 || levels[l] % 16 || levels[l] > 1024)
            return fail(LBMX_EINVAL, "unet: channels must be multiples of 16 in [16, 1024]");
    return LBMX_OK;
}

}  // namespace

extern "C" {

lbmx_status lbmx_nn_unet_workspace(const int32_t *levels, int32_t count, int32_t B, int32_t m, size_t *bytes)
{
    lbmx_status st = check_unet(levels, count, B, m);
    if (st != LBMX_OK)
        return st;
    if (!bytes)
        return fail(LBMX_EINVAL, "unet: NULL argument");
    UnetPlan plan{levels, count, B, m, nullptr, nullptr};
    st = plan.run(nullptr, nullptr, nullptr, nullptr);
    *bytes = plan.used;
    return st;
}

lbmx_status lbmx_nn_unet_forward(const float *cond, const void *const *w, const float *const *b,
                                 const int32_t *levels, int32_t count, int32_t B, int32_t m, void *ws,
                                 float *pred, void *stream)
{
    lbmx_status st = check_unet(levels, count, B, m);
    if (st != LBMX_OK)
        return st;
    if (!cond || !w || !b || !ws || !pred)
        return fail(LBMX_EINVAL, "unet: NULL argument");
    for (int k = 0; k < 4 * count - 1; ++k)
        if (!w[k])
            return fail(LBMX_EINVAL, "unet: layer %d has no weights", k);
    return UnetPlan{levels, count, B, m, stream, reinterpret_cast<char *>(ws)}.run(cond, w, b, pred);
}

lbmx_status lbmx_nn_conv3d_fwd(const void *in, const void *w, const float *bias, void *out,
                               int32_t out_f32, int32_t B, int32_t D, int32_t H, int32_t W,
                               int32_t Ci, int32_t Co, void *stream)
{
    return conv_fwd(ConvIn{reinterpret_cast<const bf *>(in), nullptr, 0}, w, bias, out, out_f32, B, D, H, W, Ci,
                    Co, stream, Epilogue{});
}

lbmx_status lbmx_nn_conv3d_fwd_ep(const void *in, const void *w, const float *bias, void *out,
                                  void *act, const void *gate, void *out2, int32_t split, int32_t B,
                                  int32_t D, int32_t H, int32_t W, int32_t Ci, int32_t Co,
                                  void *stream)
{
    Epilogue ep{reinterpret_cast<bf *>(act), reinterpret_cast<const bf *>(gate),
                reinterpret_cast<bf *>(out2), split};
    return conv_fwd(ConvIn{reinterpret_cast<const bf *>(in), nullptr, 0}, w, bias, out, 0, B, D, H, W, Ci, Co,
                    stream, ep);
}

lbmx_status lbmx_nn_conv3d_mse(const void *in, const void *w, const float *bias, const float *target,
                               int32_t K, void *grad, double *partial, int32_t npartial, float *pred,
                               int32_t B, int32_t D, int32_t H, int32_t W, int32_t Ci, int32_t Co,
                               void *stream)
{
    lbmx_status st = check_dims(B, D, H, W);
    if (st != LBMX_OK)
        return st;
    if (!in || !w || !target || !grad || !partial)
        return fail(LBMX_EINVAL, "conv3d_mse: NULL tensor");
    if (Ci < 16 || Ci % 16 || Ci > 1024 || Co < 16 || Co % 16 || Co > 1024 || K < 1 || K > Co ||
        npartial < Co / 16)
        return fail(LBMX_EINVAL, "conv3d_mse: need Ci, Co multiples of 16 in [16, 1024], 1 <= K <= Co, "
                                 "npartial >= Co / 16 (one partial per block, at least a block per "
                                 "output-channel tile)");
    const long long nvox = (long long)B * D * H * W;
    if (nvox * Co >= (1LL << 31))
        return fail(LBMX_EINVAL, "conv3d_mse: %lld voxels exceed 32-bit element indices", nvox);
    if ((st = check_plane(H, W, Ci, "conv3d_mse")) != LBMX_OK)
        return st;
    LossEp ls{target, K, 1.0f / float(double(nvox) * K), reinterpret_cast<bf *>(grad), partial, npartial};
    const ConvIn src{reinterpret_cast<const bf *>(in), nullptr, 0};
    const bf *const wb = reinterpret_cast<const bf *>(w);
    const auto run = aligned16(src.in, wb, pred, ls.grad) ? launch_fwd_as<1, 1, kLoss, 1, true>
                                                          : launch_fwd_as<1, 1, kLoss, 1, false>;
    run(src, wb, bias, pred, Dims{B, D, H, W, Ci, Co}, compute_units(), S(stream), Epilogue{}, ls);
    HIP_TRY(hipGetLastError());
    return LBMX_OK;
}

lbmx_status lbmx_nn_conv3d_fwd_upcat(const void *low, const void *skip, const void *w, const float *bias,
                                     void *out, void *act, int32_t B, int32_t D, int32_t H, int32_t W,
                                     int32_t Cu, int32_t Cs, int32_t Co, void *stream)
{
    if (!low)
        return fail(LBMX_EINVAL, "conv3d_upcat: NULL tensor");
    Epilogue ep{reinterpret_cast<bf *>(act), nullptr, nullptr, 0};
    return conv_fwd(ConvIn{reinterpret_cast<const bf *>(skip), reinterpret_cast<const bf *>(low), Cu}, w, bias,
                    out, 0, B, D, H, W, Cu + Cs, Co, stream, ep);
}

lbmx_status lbmx_nn_upcat(const void *h, const void *skip, void *cat, int32_t B, int32_t D, int32_t H,
                          int32_t W, int32_t Ch, int32_t Cs, void *stream)
{
    lbmx_status st = check_dims(B, D, H, W);
    if (st != LBMX_OK)
        return st;
    if (!h || !skip || !cat || Ch < 16 || Ch % 16 || Cs < 16 || Cs % 16)
        return fail(LBMX_EINVAL, "upcat: NULL tensor or channels not multiples of 16");
    const long long n = 8LL * B * D * H * W * ((Ch + Cs) / 8);
    if (n >= (1LL << 31))
        return fail(LBMX_EINVAL, "upcat: %lld vectors exceed 32-bit indices", n);
    hipLaunchKernelGGL(k_upcat, dim3(blocks_for(n)), dim3(256), 0, S(stream),
                       reinterpret_cast<const uint4 *>(h), reinterpret_cast<const uint4 *>(skip),
                       reinterpret_cast<uint4 *>(cat), B, D, H, W, Ch / 8, Cs / 8);
    HIP_TRY(hipGetLastError());
    return LBMX_OK;
}

lbmx_status lbmx_nn_pool2_bwd_gate(const void *gout, const void *add, const void *gate, void *gin,
                                   int32_t B, int32_t D, int32_t H, int32_t W, int32_t C, void *stream)
{
    lbmx_status st = check_dims(B, D, H, W);
    if (st != LBMX_OK)
        return st;
    if (!gout || !gin || C < 16 || C % 16 || D % 2 || H % 2 || W % 2)
        return fail(LBMX_EINVAL, "pool2_bwd_gate: NULL tensor, channels or odd extent");
    const long long n = (long long)B * D * H * W * (C / 8);
    if (n >= (1LL << 31))
        return fail(LBMX_EINVAL, "pool2_bwd_gate: %lld vectors exceed 32-bit indices", n);
    hipLaunchKernelGGL(k_pool2_bwd_gate, dim3(blocks_for(n)), dim3(256), 0, S(stream),
                       reinterpret_cast<const uint4 *>(gout), reinterpret_cast<const uint4 *>(add),
                       reinterpret_cast<const uint4 *>(gate), reinterpret_cast<uint4 *>(gin), B, D, H, W,
                       C / 8);
    HIP_TRY(hipGetLastError());
    return LBMX_OK;
}

lbmx_status lbmx_nn_up2_bwd_gate(const void *gout, const void *gate, void *gin, int32_t B, int32_t D,
                                 int32_t H, int32_t W, int32_t C, void *stream)
{
    lbmx_status st = check_dims(B, D, H, W);
    if (st != LBMX_OK)
        return st;
    if (!gout || !gin || C < 16 || C % 16)
        return fail(LBMX_EINVAL, "up2_bwd_gate: NULL tensor or channels not a multiple of 16");
    const long long n = 8LL * B * D * H * W * (C / 8);
    if (n >= (1LL << 31))
        return fail(LBMX_EINVAL, "up2_bwd_gate: %lld vectors exceed 32-bit indices", n);
    hipLaunchKernelGGL(k_up2_bwd_gate, dim3(blocks_for(n / 8)), dim3(256), 0, S(stream),
                       reinterpret_cast<const uint4 *>(gout), reinterpret_cast<const uint4 *>(gate),
                       reinterpret_cast<uint4 *>(gin), B, D, H, W, C / 8);
    HIP_TRY(hipGetLastError());
    return LBMX_OK;
}

lbmx_status lbmx_nn_conv3d_flip(const void *w, void *wt, int32_t Ci, int32_t Co, void *stream)
{
    if (!w || !wt || Ci < 1 || Co < 1)
        return fail(LBMX_EINVAL, "conv3d_flip: bad arguments");
    const long long n = (long long)Co * 27 * Ci;
    hipLaunchKernelGGL(k_conv_flip, dim3(unsigned((n + 255) / 256)), dim3(256), 0, S(stream),
                       reinterpret_cast<const bf *>(w), reinterpret_cast<bf *>(wt), Ci, Co);
    HIP_TRY(hipGetLastError());
    return LBMX_OK;
}

}  // extern "C"

namespace {

// The layer table of a flip; *most = the largest layer's element count.
lbmx_status flip_set(int32_t count, const int64_t *offsets, const int32_t *ci, const int32_t *co,
                     const char *what, FlipSet &fs, long long *most)
{
    if (!offsets || !ci || !co || count < 1 || count > FLIP_MAX)
        return fail(LBMX_EINVAL, "%s: bad layer table (1 <= count <= %d)", what, FLIP_MAX);
    fs.count = count;
    *most = 0;
    for (int l = 0; l < count; ++l) {
        if (ci[l] < 1 || co[l] < 1 || offsets[l] < 0 || (long long)co[l] * 27 * ci[l] >= (1LL << 31))
            return fail(LBMX_EINVAL, "%s: layer %d has bad shape or offset", what, l);
        fs.off[l] = offsets[l];
        fs.ci[l] = ci[l];
        fs.co[l] = co[l];
        *most = std::max(*most, (long long)co[l] * 27 * ci[l]);
    }
    return LBMX_OK;
}

}  // namespace

extern "C" {

lbmx_status lbmx_nn_conv3d_flip_many(const void *w, void *wt, int32_t count, const int64_t *offsets,
                                     const int32_t *ci, const int32_t *co, void *stream)
{
    if (!w || !wt)
        return fail(LBMX_EINVAL, "conv3d_flip_many: NULL tensor");
    FlipSet fs;
    long long most = 0;
    lbmx_status st = flip_set(count, offsets, ci, co, "conv3d_flip_many", fs, &most);
    if (st != LBMX_OK)
        return st;
    hipLaunchKernelGGL(k_conv_flip_many, dim3(blocks_for(most), unsigned(count)), dim3(256), 0, S(stream),
                       reinterpret_cast<const bf *>(w), reinterpret_cast<bf *>(wt), fs);
    HIP_TRY(hipGetLastError());
    return LBMX_OK;
}

}  // extern "C"

namespace {

lbmx_status conv_wgrad(ConvIn src, const void *gout, float *gw, float *gb, int32_t B, int32_t D, int32_t H,
                       int32_t W, int32_t Ci, int32_t Co, void *stream)
{
    lbmx_status st = check_dims(B, D, H, W);
    if (st != LBMX_OK)
        return st;
    if (!src.in || !gout || !gw)
        return fail(LBMX_EINVAL, "conv3d_wgrad: NULL tensor");
    if (Ci < 16 || Ci % 16 || Ci > 1024 || Co < 16 || Co % 16 || Co > 1024)
        return fail(LBMX_EINVAL, "conv3d_wgrad: need Ci, Co multiples of 16 in [16, 1024]");
    if ((st = check_upcat(src, D, H, W, Ci, "conv3d_wgrad")) != LBMX_OK ||
        (st = check_plane(H, W, Ci > Co ? Ci : Co, "conv3d_wgrad")) != LBMX_OK)
        return st;
    const Dims d{B, D, H, W, Ci, Co};
    const long long nv = (long long)B * D * H * W;
    if (nv * (Ci > Co ? Ci : Co) >= (1LL << 31))
        return fail(LBMX_EINVAL, "conv3d_wgrad: tensor of %lld voxels too large", nv);
    const int nbx = (W + WB_X - 1) / WB_X, nby = (H + WB_Y - 1) / WB_Y, nbz = (D + WB_Z - 1) / WB_Z;
    const long long nchunks = (long long)B * nbx * nby * nbz;
    const int pairs = (Co / 16) * (Ci / 16);
    const int cus = compute_units();
    // Blocks of one round (a block takes a whole CU, and every block adds its sums
    // to the same gradient elements) and of two chunks or more,
    // and where that costs little a multiple of 8 or 2: the blocks of all pairs that
    // read the same voxels then run on the same XCDs.  Batch 4, 160 -> 64 at 16^3 with
    // 7 blocks for each of 40 pairs, a second round of blocks, 29.6 us, with 6 19.3;
    // 32 -> 64 at 16^3 one chunk each 12.1, two 10.4.
    long long gx = std::min(std::max(1LL, (long long)cus / pairs), (nchunks + 1) / 2);
    if (gx >= 32) gx -= gx % 8;
    else if (gx >= 8) gx -= gx % 2;
    // byte offsets within a group of planes, from the voxel before its first
    const long long span = 2LL * (WB_Z + 1) * (H + 1) * (W + 2) * (Ci > Co ? Ci : Co);
    const dim3 blocks{unsigned(gx), unsigned(pairs)}, threads{64 * WB_WAVES};
    const bf *const g = reinterpret_cast<const bf *>(gout);
    if (span < (long long)kRange && aligned16(src.in, src.low, g))
        hipLaunchKernelGGL(k_conv_wgrad<true>, blocks, threads, 0, S(stream), src, g, gw, gb, d, nbx, nby, nbz);
    else
        hipLaunchKernelGGL(k_conv_wgrad<false>, blocks, threads, 0, S(stream), src, g, gw, gb, d, nbx, nby, nbz);
    HIP_TRY(hipGetLastError());
    return LBMX_OK;
}

}  // namespace

extern "C" {

lbmx_status lbmx_nn_conv3d_wgrad(const void *in, const void *gout, float *gw, float *gb, int32_t B,
                                 int32_t D, int32_t H, int32_t W, int32_t Ci, int32_t Co, void *stream)
{
    return conv_wgrad(ConvIn{reinterpret_cast<const bf *>(in), nullptr, 0}, gout, gw, gb, B, D, H, W, Ci, Co,
                      stream);
}

lbmx_status lbmx_nn_conv3d_wgrad_upcat(const void *low, const void *skip, const void *gout, float *gw,
                                       float *gb, int32_t B, int32_t D, int32_t H, int32_t W, int32_t Cu,
                                       int32_t Cs, int32_t Co, void *stream)
{
    if (!low)
        return fail(LBMX_EINVAL, "conv3d_wgrad_upcat: NULL tensor");
    return conv_wgrad(ConvIn{reinterpret_cast<const bf *>(skip), reinterpret_cast<const bf *>(low), Cu}, gout,
                      gw, gb, B, D, H, W, Cu + Cs, Co, stream);
}

lbmx_status lbmx_nn_silu(const void *z, void *a, int64_t n, void *stream)
{
    if (!z || !a || n < 0)
        return fail(LBMX_EINVAL, "silu: bad arguments");
    hipLaunchKernelGGL(k_silu_fwd, dim3(blocks_for(n)), dim3(256), 0, S(stream),
                       reinterpret_cast<const bf *>(z), reinterpret_cast<bf *>(a), (long long)n);
    HIP_TRY(hipGetLastError());
    return LBMX_OK;
}

lbmx_status lbmx_nn_silu_bwd(const void *z, const void *ga, void *gz, int64_t n, void *stream)
{
    if (!z || !ga || !gz || n < 0)
        return fail(LBMX_EINVAL, "silu_bwd: bad arguments");
    hipLaunchKernelGGL(k_silu_bwd, dim3(blocks_for(n)), dim3(256), 0, S(stream),
                       reinterpret_cast<const bf *>(z), reinterpret_cast<const bf *>(ga),
                       reinterpret_cast<bf *>(gz), (long long)n);
    HIP_TRY(hipGetLastError());
    return LBMX_OK;
}

lbmx_status lbmx_nn_pool2(const void *in, void *out, int32_t B, int32_t D, int32_t H, int32_t W,
                          int32_t C, int32_t backward, void *stream)
{
    lbmx_status st = check_dims(B, D, H, W);
    if (st != LBMX_OK)
        return st;
    if (!in || !out || C < 1 || D % 2 || H % 2 || W % 2)
        return fail(LBMX_EINVAL, "pool2: need even extents");
    const long long n = (long long)B * D * H * W * C;
    if (backward)  // in = gradient of the pooled tensor, out = gradient of the input
        hipLaunchKernelGGL(k_pool2_bwd, dim3(blocks_for(n)), dim3(256), 0, S(stream),
                           reinterpret_cast<const bf *>(in), reinterpret_cast<bf *>(out), B, D, H, W, C);
    else if (C % 8 == 0 && n < (1LL << 31))
        hipLaunchKernelGGL(k_pool2_fwd8, dim3(blocks_for(n / 64)), dim3(256), 0, S(stream),
                           reinterpret_cast<const uint4 *>(in), reinterpret_cast<uint4 *>(out), B, D, H, W,
                           C / 8);
    else
        hipLaunchKernelGGL(k_pool2_fwd, dim3(blocks_for(n / 8)), dim3(256), 0, S(stream),
                           reinterpret_cast<const bf *>(in), reinterpret_cast<bf *>(out), B, D, H, W, C);
    HIP_TRY(hipGetLastError());
    return LBMX_OK;
}

lbmx_status lbmx_nn_up2(const void *in, void *out, int32_t B, int32_t D, int32_t H, int32_t W,
                        int32_t C, int32_t backward, void *stream)
{
    lbmx_status st = check_dims(B, D, H, W);
    if (st != LBMX_OK)
        return st;
    if (!in || !out || C < 1)
        return fail(LBMX_EINVAL, "up2: bad arguments");
    const long long n = (long long)B * D * H * W * C;
    if (backward)  // in = gradient of the upsampled tensor, out = gradient of the input
        hipLaunchKernelGGL(k_up2_bwd, dim3(blocks_for(n)), dim3(256), 0, S(stream),
                           reinterpret_cast<const bf *>(in), reinterpret_cast<bf *>(out), B, D, H, W, C);
    else
        hipLaunchKernelGGL(k_up2_fwd, dim3(blocks_for(8 * n)), dim3(256), 0, S(stream),
                           reinterpret_cast<const bf *>(in), reinterpret_cast<bf *>(out), B, D, H, W, C);
    HIP_TRY(hipGetLastError());
    return LBMX_OK;
}

lbmx_status lbmx_nn_concat(void *a, void *b, void *out, int64_t nvox, int32_t Ca, int32_t Cb,
                           int32_t backward, void *stream)
{
    if (!a || !b || !out || nvox < 0 || Ca < 1 || Cb < 1)
        return fail(LBMX_EINVAL, "concat: bad arguments");
    const long long n = (long long)nvox * (Ca + Cb);
    if (backward)  // out = gradient of the concatenation, a / b receive the parts
        hipLaunchKernelGGL(k_split, dim3(blocks_for(n)), dim3(256), 0, S(stream),
                           reinterpret_cast<const bf *>(out), reinterpret_cast<bf *>(a),
                           reinterpret_cast<bf *>(b), (long long)nvox, Ca, Cb);
    else
        hipLaunchKernelGGL(k_concat, dim3(blocks_for(n)), dim3(256), 0, S(stream),
                           reinterpret_cast<const bf *>(a), reinterpret_cast<const bf *>(b),
                           reinterpret_cast<bf *>(out), (long long)nvox, Ca, Cb);
    HIP_TRY(hipGetLastError());
    return LBMX_OK;
}

lbmx_status lbmx_nn_mse(const float *pred, const float *target, void *grad, double *partial,
                        int32_t npartial, int64_t nvox, int32_t C, int32_t K, void *stream)
{
    if (!pred || !target || !grad || !partial || npartial < 1 || npartial > 4096 || K < 1 || K > C)
        return fail(LBMX_EINVAL, "mse: bad arguments");
    const float scale = 1.0f / float(double(nvox) * K);
    if (C % 8 == 0 && K <= 8)
        hipLaunchKernelGGL(k_mse_v, dim3(npartial), dim3(256), 0, S(stream), pred, target,
                           reinterpret_cast<uint4 *>(grad), partial, (long long)nvox, C, K, scale);
    else
        hipLaunchKernelGGL(k_mse, dim3(npartial), dim3(256), 0, S(stream), pred, target,
                           reinterpret_cast<bf *>(grad), partial, (long long)nvox, C, K, scale);
    HIP_TRY(hipGetLastError());
    return LBMX_OK;
}

lbmx_status lbmx_nn_adam(float *w, float *g, float *m, float *v, void *w_bf16, int64_t n, float lr,
                         float b1, float b2, float eps, int64_t step, float wd, void *stream)
{
    if (!w || !g || !m || !v || n < 0 || step < 1)
        return fail(LBMX_EINVAL, "adam: bad arguments");
    const float c1 = float(1.0 / (1.0 - std::pow(double(b1), double(step))));
    const float c2 = float(1.0 / (1.0 - std::pow(double(b2), double(step))));
    hipLaunchKernelGGL(k_adam, dim3(blocks_for(n)), dim3(256), 0, S(stream), w, g, m, v,
                       reinterpret_cast<bf *>(w_bf16), (long long)n, lr, b1, b2, eps, c1, c2, wd,
                       static_cast<bf *>(nullptr), FlipSet{});
    HIP_TRY(hipGetLastError());
    return LBMX_OK;
}

lbmx_status lbmx_nn_adam_flip(float *w, float *g, float *m, float *v, void *w_bf16, void *w_flip,
                              int64_t n, float lr, float b1, float b2, float eps, int64_t step, float wd,
                              int32_t count, const int64_t *offsets, const int32_t *ci, const int32_t *co,
                              void *stream)
{
    if (!w || !g || !m || !v || !w_bf16 || !w_flip || n < 0 || step < 1)
        return fail(LBMX_EINVAL, "adam_flip: bad arguments");
    FlipSet fs;
    long long most = 0;
    lbmx_status st = flip_set(count, offsets, ci, co, "adam_flip", fs, &most);
    if (st != LBMX_OK)
        return st;
    for (int l = 0; l < count; ++l)
        if ((l > 0 && offsets[l] < offsets[l - 1] + (long long)co[l - 1] * 27 * ci[l - 1]) ||
            offsets[l] + (long long)co[l] * 27 * ci[l] > n)
            return fail(LBMX_EINVAL, "adam_flip: layers overlap, are not ascending or exceed n");
    const float c1 = float(1.0 / (1.0 - std::pow(double(b1), double(step))));
    const float c2 = float(1.0 / (1.0 - std::pow(double(b2), double(step))));
    hipLaunchKernelGGL(k_adam, dim3(blocks_for(n)), dim3(256), 0, S(stream), w, g, m, v,
                       reinterpret_cast<bf *>(w_bf16), (long long)n, lr, b1, b2, eps, c1, c2, wd,
                       reinterpret_cast<bf *>(w_flip), fs);
    HIP_TRY(hipGetLastError());
    return LBMX_OK;
}

lbmx_status lbmx_nn_to_bf16(const float *a, void *b, int64_t n, void *stream)
{
    if (!a || !b || n < 0)
        return fail(LBMX_EINVAL, "to_bf16: bad arguments");
    hipLaunchKernelGGL(k_f32_to_bf16, dim3(blocks_for(n)), dim3(256), 0, S(stream), a,
                       reinterpret_cast<bf *>(b), (long long)n);
    HIP_TRY(hipGetLastError());
    return LBMX_OK;
}

lbmx_status lbmx_nn_make_input(const float *cond, void *out, int32_t B, int32_t m, void *stream)
{
    if (!cond || !out || B < 1 || m < 1 || (long long)B * m * m >= (1LL << 31))
        return fail(LBMX_EINVAL, "make_input: bad arguments (B m^2 < 2^31 rows)");
    hipLaunchKernelGGL(k_make_input, dim3(unsigned(B * m * m)), dim3(128), 0, S(stream), cond,
                       reinterpret_cast<bf *>(out), m);
    HIP_TRY(hipGetLastError());
    return LBMX_OK;
}

lbmx_status lbmx_nn_add(const void *a, const void *b, void *out, int64_t n, void *stream)
{
    if (!a || !b || !out || n < 0)
        return fail(LBMX_EINVAL, "add: bad arguments");
    hipLaunchKernelGGL(k_add, dim3(blocks_for(n)), dim3(256), 0, S(stream), reinterpret_cast<const bf *>(a),
                       reinterpret_cast<const bf *>(b), reinterpret_cast<bf *>(out), (long long)n);
    HIP_TRY(hipGetLastError());
    return LBMX_OK;
}

lbmx_status lbmx_nn_layout_flip(const float *a, float *b, int32_t B, int32_t m, int32_t K, int32_t C,
                                int32_t flip, const float *signs, const float *scale, void *stream)
{
    if (!a || !b || B < 1 || m < 1 || K < 1 || K > 8 || K > C || flip < 0 || flip > 7 || !signs)
        return fail(LBMX_EINVAL, "layout_flip: bad arguments (1 <= K <= min(C, 8), 0 <= flip <= 7)");
    ChannelSigns sg{};
    for (int k = 0; k < K; ++k)
        sg.s[k] = signs[k];
    const long long n = (long long)B * m * m * m * C;
    hipLaunchKernelGGL(k_cf_to_cl_flip, dim3(blocks_for(n)), dim3(256), 0, S(stream), a, b, B, m, K, C, flip,
                       sg, scale);
    HIP_TRY(hipGetLastError());
    return LBMX_OK;
}

lbmx_status lbmx_nn_layout(const float *a, float *b, int32_t B, int64_t V, int32_t K, int32_t C,
                           int32_t to_channel_last, const float *scale, void *stream)
{
    if (!a || !b || B < 1 || V < 1 || K < 1 || K > C)
        return fail(LBMX_EINVAL, "layout: bad arguments");
    if (to_channel_last) {
        const long long n = (long long)B * V * C;
        hipLaunchKernelGGL(k_cf_to_cl, dim3(blocks_for(n)), dim3(256), 0, S(stream), a, b, B,
                           (long long)V, K, C, scale);
    } else {
        const long long n = (long long)B * V * K;
        hipLaunchKernelGGL(k_cl_to_cf, dim3(blocks_for(n)), dim3(256), 0, S(stream), a, b, B,
                           (long long)V, K, C, scale);
    }
    HIP_TRY(hipGetLastError());
    return LBMX_OK;
}

}  // extern "C"
