// gfx950 kernels of the spatially split VAE tile (paper Sec. 3.6): the
// causal 3D convolutions of a VAE stage run on each tile's region (its core
// widened by a halo), and the blended gather of the tiles into the plane.
//
// Convolution as an implicit GEMM on the four-wave MFMA tile kernel
// (gemm_tile.hpp): rows are the output pixels (tile, frame, row, column) of
// the listed tiles, K runs over the 27 taps x Cin channels, and the weights
// [Cout, 3, 3, 3, Cin] are K-contiguous per output channel -- the linear
// layer's layout.  Channels-last activations make every (pixel, tap) a
// contiguous run of Cin values, so a K step of 64 channels of one tap is
// one 128-byte row per pixel, copied HBM -> LDS like a dense row; a tap
// that falls before the first frame or outside the tile's region is copied
// from a page of zeros instead (the zero padding).  Where the output tiles are
// too few to fill the compute units (one GPU's single tile), K is split into
// ranges whose f32 partial sums a second kernel adds, with the bias and the
// activation.
//
// Blend: one thread per (pixel, 8 channels) walks the tiles whose region
// covers the pixel and adds weight x value, the weight the product of the
// two axes' ramps (fp32).  HBM-bound.
#include "vae_kernels.hpp"

#include <stdint.h>

#include <algorithm>

#include "attn_kernels.hpp"
#include "gemm_tile.hpp"
#include "tile_plan.hpp"

// 128 bytes of zeros in device memory: the source of the copies that stand
// for padding taps (read only).
static __device__ __align__(256) uint16_t vae_zero_page[64] = {0};

namespace regenvc {
namespace {

using tile::kBK;

typedef tile::bf16x8 bf16x8;
typedef tile::f32x4 f32x4;

typedef tile::Shape4<8, 8, 3, 1> Tile256x256;
typedef tile::Shape4<8, 6, 3, 1> Tile256x192;
typedef tile::Shape4<6, 6, 3, 1> Tile192x192;
typedef tile::Shape4<4, 6, 3, 1> Tile128x192;
typedef tile::Shape4<4, 4, 3, 2> Tile128x128;

enum ConvTile : int32_t { kConv256x256, kConv256x192, kConv192x192, kConv128x192, kConv128x128 };

// n / d and n % d for n < 2^31 with inv = min(2^32 / d, 2^32 - 1): the
// estimate is at most one too small.
__device__ __forceinline__ int div_by(int n, int d, uint32_t inv, int &rem)
{
    int q = (int)__umulhi((uint32_t)n, inv);
    rem = n - q * d;
    if (rem >= d) rem -= d, ++q;
    return q;
}

// K of the convolution runs over the channels in blocks of 64 and, within a
// block, over the 27 taps: K step kt = channels 64 (kt / 27) .. +63 of tap
// kt % 27.  A pixel's 128 bytes of a block are then read again by the
// neighbouring taps one, three and nine steps later, while they are still in
// the XCD's L2 (the 32 tiles of an XCD read 1 MB of pixels a step); with the
// taps outermost they came from beyond it.
constexpr int kTaps = 27;

// Input channels from which the offsets within a tile's weight rows (255 rows
// of 27 Cin elements) may leave 32 bits.
constexpr int kWideCin = (1 << 22) / kTaps + 1;

// Weight rows [27, Cin] in that order.
template <bool WIDE>
struct ConvW : tile::Dense<WIDE> {
    int Cin;
    typedef typename tile::Dense<WIDE>::Step Step;
    __device__ Step at(int kt) const
    {
        const int c = (int)((uint32_t)kt / kTaps), tap = kt - c * kTaps;
        Step s = tile::Dense<WIDE>::at(c);
        s.base += (int64_t)tap * (Cin * 2);
        return s;
    }
};

// A rows of the convolution: pixel m of the listed tiles' regions.  A row keeps
// the address of its own pixel (the centre tap of the current frame) and one
// bit per tap that is set where the tap lies inside the region; what depends
// on the tap alone is wave-uniform (scalar).  A copy then costs a select
// between the tap's address and the page of zeros, without a branch.
struct ConvSrc {
    const ConvArgs *a;
    int m0, rows;
    struct Row {
        const char *ptr;
        uint32_t ok;
    };
    __device__ Row row(int r, int chunk) const
    {
        int x, y, t;
        const int m = min(m0 + r, rows - 1);
        int q = div_by(m, a->Wr, a->inv_w, x);
        q = div_by(q, a->Hr, a->inv_h, y);
        const int ti = div_by(q, a->T, a->inv_t, t);
        const VaeTile &tl = a->tiles[ti];
        const int h = tl.reg_y1 - tl.reg_y0, w = tl.reg_x1 - tl.reg_x0;
        int64_t pix;
        if (a->in_is_plane)
            pix = ((int64_t)t * a->H + tl.reg_y0 + y) * a->W + tl.reg_x0 + x;
        else
            pix = (((int64_t)ti * a->T + t) * a->Hr + y) * a->Wr + x;
        Row o;
        o.ptr = static_cast<const char *>(a->in) + pix * a->Cin * 2 + chunk * 16;
        // taps dx = -1, 0, 1 as bits 0..2, then three rows of them, then three frames
        uint32_t bx = 0, by = 0;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            if ((unsigned)(x + d - 1) < (unsigned)w) bx |= 1u << d;
        }
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            if ((unsigned)(y + d - 1) < (unsigned)h) by |= bx << (3 * d);
        }
        o.ok = by << 18;
        if (t >= 1) o.ok |= by << 9;
        if (t >= 2) o.ok |= by;
        return o;
    }
    // The tap of K step kt: its offset from a row's own pixel and its bit.  Lane
    // l of tap_lo, tap_hi holds the offset of tap l: read from there, a step's
    // scalar work is a dozen instructions (forming the offset takes forty, which
    // one wave per SIMD cannot hide).
    struct Step {
        uint32_t lo, hi, bit;
    };
    uint32_t tap_lo, tap_hi;
    __device__ void init()
    {
        const int tap = (int)threadIdx.x & 31;
        const int64_t off = a->tap0 + (int64_t)tap * (a->Cin * 2) + (int64_t)(tap / 3) * a->row_jump +
                            (int64_t)(tap / 9) * a->frame_jump;
        tap_lo = (uint32_t)off, tap_hi = (uint32_t)((uint64_t)off >> 32);
    }
    __device__ Step at(int kt) const
    {
        const uint32_t c = (uint32_t)kt / kTaps, tap = (uint32_t)kt - c * kTaps;
        const uint64_t off = (((uint64_t)(uint32_t)__builtin_amdgcn_readlane(tap_hi, tap) << 32) |
                              (uint32_t)__builtin_amdgcn_readlane(tap_lo, tap)) + (uint64_t)c * tile::kRowBytes;
        return Step{(uint32_t)off, (uint32_t)(off >> 32), 1u << tap};
    }
    struct Addr {
        const void *ptr;
    };
    __device__ Addr addr(const Row &r, const Step &s) const
    {
        const uint64_t p = reinterpret_cast<uint64_t>(r.ptr) + (((uint64_t)s.hi << 32) | s.lo);
        const uint64_t z = reinterpret_cast<uint64_t>(static_cast<const void *>(vae_zero_page));
        const bool ok = (r.ok & s.bit) != 0;
        const uint32_t lo = ok ? (uint32_t)p : (uint32_t)z, hi = ok ? (uint32_t)(p >> 32) : (uint32_t)(z >> 32);
        return Addr{reinterpret_cast<const void *>(((uint64_t)hi << 32) | lo)};
    }
    __device__ void copy(const Addr &ad, uint32_t lds) const { tile::lds_copy16_v(ad.ptr, lds); }
};

// One tile of shape S per workgroup.  EPI == kPartial: split-K, f32 partial
// sums of `splits` K ranges into the workspace (bias and activation follow in
// vae_reduce_kernel).
template <class S, int EPI, bool WIDE>
__global__ __launch_bounds__(tile::kThreads4) __attribute__((amdgpu_waves_per_eu(S::WPE, S::WPE)))
void conv3d_kernel(ConvArgs a, int tiles_n, int n_tiles, int splits)
{
    __shared__ __attribute__((aligned(1024))) char smem[S::LDS];
    constexpr bool PART = EPI == tile::kPartial;
    const int sp = PART ? (int)blockIdx.x / n_tiles : 0;
    int tm, tn;
    tile::tile_of((int)blockIdx.x - sp * n_tiles, tiles_n, n_tiles, tm, tn);
    const int m0 = tm * S::BM, n0 = tn * S::BN;
    const int nk = kTaps * (a.Cin / kBK), M = a.n_tiles * a.T * a.Hr * a.Wr;
    const int k0 = PART ? (int)((int64_t)sp * nk / splits) : 0;
    const int k1 = PART ? (int)((int64_t)(sp + 1) * nk / splits) : nk;
    ConvSrc as{&a, m0, M};
    as.init();
    const ConvW<WIDE> ws{{static_cast<const uint16_t *>(a.w), (int64_t)kTaps * a.Cin, a.Cout, n0}, a.Cin};
    f32x4 acc[S::NB][S::MB];
    tile::mma4<S>(as, ws, k0, k1, smem, acc);
    const tile::Out o{static_cast<const uint16_t *>(a.bias), nullptr, PART ? a.ws : a.out, a.Cout, M, a.Cout};
    tile::store4<S, EPI>(o, m0, n0, sp, smem, acc);
}

// Sum of the split-K partials, bias and activation: one thread per 8
// channels of one output row.
template <bool SILU>
__global__ __launch_bounds__(256) void vae_reduce_kernel(ConvArgs a, int splits)
{
    const int64_t M = (int64_t)a.n_tiles * a.T * a.Hr * a.Wr;
    const int cg = a.Cout / 8;
    const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (gid >= M * cg) return;
    const int64_t m = gid / cg;
    const int c = (int)(gid - m * cg) * 8;
    const float *p = static_cast<const float *>(a.ws) + m * a.Cout + c;
    f32x4 s0 = *reinterpret_cast<const f32x4 *>(p), s1 = *reinterpret_cast<const f32x4 *>(p + 4);
    for (int k = 1; k < splits; ++k) {
        const float *q = p + (int64_t)k * M * a.Cout;
        s0 += *reinterpret_cast<const f32x4 *>(q);
        s1 += *reinterpret_cast<const f32x4 *>(q + 4);
    }
    const bf16x8 bb = *reinterpret_cast<const bf16x8 *>(static_cast<const uint16_t *>(a.bias) + c);
    bf16x8 o;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float y = (e < 4 ? s0[e] : s1[e - 4]) + (float)bb[e];
        o[e] = (__bf16)(SILU ? tile::silu(y) : y);
    }
    *reinterpret_cast<bf16x8 *>(static_cast<uint16_t *>(a.out) + m * a.Cout + c) = o;
}

__device__ __forceinline__ float ramp(int p, int c0, int c1, int n, int band)
{
    if (band == 0) return (p >= c0 && p < c1) ? 1.f : 0.f;
    const float pc = (float)p + 0.5f, inv = 0.5f / (float)band;
    float w = 1.f;
    if (c0 > 0) w = fminf(w, fminf(fmaxf(((float)band + (pc - (float)c0)) * inv, 0.f), 1.f));
    if (c1 < n) w = fminf(w, fminf(fmaxf(((float)band + ((float)c1 - pc)) * inv, 0.f), 1.f));
    return w;
}

__global__ __launch_bounds__(256) void vae_blend_kernel(BlendArgs a)
{
    const int cg = a.C / 8;
    const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (gid >= (int64_t)a.T * a.H * a.W * cg) return;
    const int c = (int)(gid % cg) * 8;
    int64_t q = gid / cg;
    const int x = (int)(q % a.W);
    q /= a.W;
    const int y = (int)(q % a.H);
    const int t = (int)(q / a.H);
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    const uint16_t *src = static_cast<const uint16_t *>(a.tiles_out);
    for (int i = 0; i < a.n_tiles; ++i) {
        const VaeTile &tl = a.tiles[i];
        if (y < tl.reg_y0 || y >= tl.reg_y1 || x < tl.reg_x0 || x >= tl.reg_x1) continue;
        const float w = ramp(y, tl.core_y0, tl.core_y1, a.H, a.band) * ramp(x, tl.core_x0, tl.core_x1, a.W, a.band);
        if (w == 0.f) continue;
        const int64_t pix = (((int64_t)i * a.T + t) * a.Hr + (y - tl.reg_y0)) * a.Wr + (x - tl.reg_x0);
        const bf16x8 v = *reinterpret_cast<const bf16x8 *>(src + pix * a.C + c);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] = fmaf(w, (float)v[e], acc[e]);
    }
    bf16x8 o;
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = (__bf16)acc[e];
    *reinterpret_cast<bf16x8 *>(static_cast<uint16_t *>(a.out) + (((int64_t)t * a.H + y) * a.W + x) * a.C + c) = o;
}

template <class S, bool WIDE = false>
hipError_t launch_conv(const ConvArgs &a, int splits, hipStream_t stream)
{
    const int64_t M = (int64_t)a.n_tiles * a.T * a.Hr * a.Wr;
    const int tiles_n = tile::tiles_along(a.Cout, S::BN);
    const int n_tiles = (int)((M + S::BM - 1) / S::BM) * tiles_n;
    const dim3 grid((unsigned)n_tiles * (unsigned)splits), block(tile::kThreads4);
    if (splits > 1) {
        hipLaunchKernelGGL((conv3d_kernel<S, tile::kPartial, WIDE>), grid, block, 0, stream, a, tiles_n, n_tiles, splits);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        const int64_t n = M * (a.Cout / 8);
        const dim3 rgrid((unsigned)((n + 255) / 256));
        if (a.silu)
            hipLaunchKernelGGL(vae_reduce_kernel<true>, rgrid, dim3(256), 0, stream, a, splits);
        else
            hipLaunchKernelGGL(vae_reduce_kernel<false>, rgrid, dim3(256), 0, stream, a, splits);
    } else if (a.silu) {
        hipLaunchKernelGGL((conv3d_kernel<S, tile::kBiasSilu, WIDE>), grid, block, 0, stream, a, tiles_n, n_tiles, 1);
    } else {
        hipLaunchKernelGGL((conv3d_kernel<S, tile::kBias, WIDE>), grid, block, 0, stream, a, tiles_n, n_tiles, 1);
    }
    return hipGetLastError();
}

}  // namespace

// The tile and K split of a convolution, by plan_tiles with constants fitted to
// timed launches.  Over 110 shapes of 320 to 174720 pixels and 64 to 512
// channels, each timed on every tile and split, the choice is on average 1.2 %
// slower than the best, at most 18 % (43680 pixels x 256 -> 128 channels, 97 us
// on 192 x 192, 82 on 128 x 128).  64736 pixels x 384 channels: 416-420 ->
// 362-370 us a convolution (256 x 192, 506 tiles: two rounds); one tile of the
// split plane (8092 pixels) 68.0 + 9.2 -> 68.7 + 6.4 us with the second kernel
// (128 x 192 in two ranges, where four wrote twice the partial sums).  A step
// costs a fifth more than a linear layer's: its pixel addresses are selected in
// vector registers.
TilePlan conv_plan(int64_t M, int N, int Cin, int n_cu, int64_t ws_bytes)
{
    static const TileCost kCosts[] = {
        {kConv256x256, 256, 256, 4, 15.0, 15.0, 1.20, 1.15, true},
        {kConv256x192, 256, 192, 4, 12.2, 12.2, 0.947, 1.15, true},
        {kConv192x192, 192, 192, 4, 10.9, 10.9, 0.75, 1.15, true},
        {kConv128x192, 128, 192, 4, 7.6, 7.6, 0.569, 1.15, true},
        {kConv128x128, 128, 128, 4, 2.0, 2.0, 0.45, 1.05, true},
    };
    const SplitCost split{3.0, 7.0e6, 2};
    const int nk = kTaps * (Cin / kBK);
    if (Cin >= kWideCin) {  // the one tile that such weight rows have
        const TileCost wide[] = {kCosts[4]};
        return plan_tiles(wide, split, M, N, nk, n_cu, ws_bytes);
    }
    return plan_tiles(kCosts, split, M, N, nk, n_cu, ws_bytes);
}

size_t conv_workspace_bytes(int64_t M, int N, int Cin, int n_cu)
{
    const int s = conv_plan(M, N, Cin, n_cu, INT64_MAX).splits;
    return s > 1 ? (size_t)s * M * N * sizeof(float) : 0;
}

hipError_t launch_vae_conv(const ConvArgs &args, hipStream_t stream)
{
    const int64_t M = (int64_t)args.n_tiles * args.T * args.Hr * args.Wr;
    if (M == 0) return hipSuccess;
    ConvArgs a = args;
    auto inv = [](int d) { return (uint32_t)std::min<uint64_t>((1ull << 32) / (uint32_t)d, 0xffffffffu); };
    a.inv_w = inv(a.Wr), a.inv_h = inv(a.Hr), a.inv_t = inv(a.T);
    const int64_t px = (int64_t)a.Cin * 2, row = (a.in_is_plane ? a.W : a.Wr) * px;
    const int64_t frame = (a.in_is_plane ? a.H : a.Hr) * row;
    a.tap0 = -2 * frame - row - px;  // tap (-2, -1, -1)
    a.row_jump = row - 3 * px, a.frame_jump = frame - 3 * row;
    const TilePlan p = conv_plan(M, a.Cout, a.Cin, device_cu_count(), a.ws != nullptr ? a.ws_bytes : 0);
    if (a.Cin >= kWideCin) return launch_conv<Tile128x128, true>(a, p.splits, stream);
    switch (p.tile) {
    case kConv256x256: return launch_conv<Tile256x256>(a, p.splits, stream);
    case kConv256x192: return launch_conv<Tile256x192>(a, p.splits, stream);
    case kConv192x192: return launch_conv<Tile192x192>(a, p.splits, stream);
    case kConv128x192: return launch_conv<Tile128x192>(a, p.splits, stream);
    case kConv128x128: return launch_conv<Tile128x128>(a, p.splits, stream);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_vae_blend(const BlendArgs &a, hipStream_t stream)
{
    const int64_t n = (int64_t)a.T * a.H * a.W * (a.C / 8);
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(vae_blend_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, a);
    return hipGetLastError();
}

}  // namespace regenvc
