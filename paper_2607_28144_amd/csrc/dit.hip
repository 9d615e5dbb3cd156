// gfx950 kernels of the diffusion-transformer block around the attention:
// linear layers (bf16 MFMA, fp32 accumulation) with the block's pointwise
// work fused into their epilogues, the layer normalizations with the adaLN
// modulation, the row RMSNorm of the cross-attention query and the adaLN
// modulation vectors.
//
// Linear layer y = a W^T, a [M, K] and W [N, K] both K-contiguous (the weight
// layout of a linear layer): the bf16 MFMA tile kernels of gemm_tile.hpp with
// dense rows, four waves per tile of 64 x 128 to 256 x 256 or eight per
// 256 x 256 and 288 x 256, K split over workgroups where the tiles are few
// (linear_plan).
#include "dit_kernels.hpp"

#include "attn_kernels.hpp"
#include "gemm_tile.hpp"
#include "tile_plan.hpp"

namespace regenvc {
namespace {

using tile::bf;
using tile::kBK;
using tile::kThreads;
typedef tile::bf16x8 bf16x8;
typedef tile::f32x4 f32x4;

// Linear layer, one BM x 256 tile per workgroup of eight waves.
template <int BM, int EPI>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void linear_kernel(LinearArgs a, int tiles_n, int n_tiles)
{
    __shared__ __attribute__((aligned(1024))) char smem[tile::lds_bytes<BM>()];
    const tile::Out o{static_cast<const uint16_t *>(a.bias), a.gate, a.out, a.ldo, a.M, a.N};
    tile::tile_body<BM, EPI>(static_cast<const uint16_t *>(a.a), a.lda, static_cast<const uint16_t *>(a.w), a.K, o,
                             tiles_n, n_tiles, smem);
}

// Four-wave tiles of a linear layer.
typedef tile::Shape4<8, 8, 3, 1> Tile256x256;
typedef tile::Shape4<5, 8, 3, 1> Tile160x256;
typedef tile::Shape4<6, 6, 3, 1> Tile192x192;
typedef tile::Shape4<4, 4, 3, 2> Tile128x128;
typedef tile::Shape4<2, 4, 2, 3> Tile64x128;
typedef tile::Shape4<4, 6, 3, 1> Tile128x192;

// Row strides from which the offsets within a tile (255 rows) may leave 32 bits.
constexpr int64_t kWideStride = 1 << 22;

// Linear layer, one tile of shape S per workgroup of four waves.  EPI ==
// kPartial: K range blockIdx.x / n_tiles of `splits`, f32 sums to its
// [M][N] plane of the workspace.
template <class S, int EPI, bool WIDE>
__global__ __launch_bounds__(tile::kThreads4) __attribute__((amdgpu_waves_per_eu(S::WPE, S::WPE)))
void linear4_kernel(LinearArgs a, int tiles_n, int n_tiles, int splits)
{
    __shared__ __attribute__((aligned(1024))) char smem[S::LDS];
    constexpr bool PART = EPI == tile::kPartial;
    const int sp = PART ? (int)blockIdx.x / n_tiles : 0;
    int tm, tn;
    tile::tile_of((int)blockIdx.x - sp * n_tiles, tiles_n, n_tiles, tm, tn);
    const int m0 = tm * S::BM, n0 = tn * S::BN;
    const int nk = a.K / kBK;
    const int k0 = PART ? (int)((int64_t)sp * nk / splits) : 0;
    const int k1 = PART ? (int)((int64_t)(sp + 1) * nk / splits) : nk;
    const tile::Dense<WIDE> as{static_cast<const uint16_t *>(a.a), a.lda, a.M, m0};
    const tile::Dense<WIDE> ws{static_cast<const uint16_t *>(a.w), a.K, a.N, n0};
    f32x4 acc[S::NB][S::MB];
    if (k1 > k0) {
        tile::mma4<S>(as, ws, k0, k1, smem, acc);
    } else {
#pragma unroll
        for (int nb = 0; nb < S::NB; ++nb)
#pragma unroll
            for (int mb = 0; mb < S::MB; ++mb) acc[nb][mb] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const tile::Out o{static_cast<const uint16_t *>(a.bias), a.gate, PART ? a.ws : a.out, PART ? (int64_t)a.N : a.ldo,
                      a.M, a.N};
    tile::store4<S, EPI>(o, m0, n0, sp, smem, acc);
}

// Sum of the split-K partials and the epilogue: one thread per 8 channels of
// one row.
template <int EPI>
__global__ __launch_bounds__(256) void linear_reduce_kernel(LinearArgs a, int splits)
{
    const int cg = a.N / 8;
    const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (gid >= (int64_t)a.M * cg) return;
    const int64_t m = gid / cg;
    const int n = (int)(gid - m * cg) * 8;
    const float *p = a.ws + m * a.N + n;
    const int64_t plane = (int64_t)a.M * a.N;
    f32x4 s[2] = {*reinterpret_cast<const f32x4 *>(p), *reinterpret_cast<const f32x4 *>(p + 4)};
    for (int k = 1; k < splits; ++k) {
        s[0] += *reinterpret_cast<const f32x4 *>(p + k * plane);
        s[1] += *reinterpret_cast<const f32x4 *>(p + k * plane + 4);
    }
    s[0] += tile::load_bias4(static_cast<const uint16_t *>(a.bias), n);
    s[1] += tile::load_bias4(static_cast<const uint16_t *>(a.bias), n + 4);
    if constexpr (EPI == kEpiGatedRes) {
        f32x4 *q = reinterpret_cast<f32x4 *>(static_cast<float *>(a.out) + m * a.ldo + n);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const f32x4 gv = a.gate != nullptr ? *reinterpret_cast<const f32x4 *>(a.gate + n + 4 * h)
                                               : f32x4{1.f, 1.f, 1.f, 1.f};
            q[h] = q[h] + gv * s[h];
        }
    } else {
        bf16x8 o;
#pragma unroll
        for (int i = 0; i < 8; ++i) o[i] = (__bf16)tile::activate<EPI>(s[i / 4][i % 4]);
        *reinterpret_cast<bf16x8 *>(static_cast<uint16_t *>(a.out) + m * a.ldo + n) = o;
    }
}

// ---------------------------------------------------------------- row norms
__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
    return v;
}

// One wave per row of C = 512 * NCH channels; lane l holds channels
// 512 j + 8 l .. +7 for j < NCH.  Two-pass mean and variance in registers.
template <int NCH>
__global__ __launch_bounds__(256) void layer_norm_kernel(LayerNormArgs a)
{
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= a.rows) return;
    const float *xr = a.x + row * a.ldx;
    f32x4 v[NCH][2];
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < NCH; ++j) {
        const int c = 512 * j + 8 * lane;
        v[j][0] = *reinterpret_cast<const f32x4 *>(xr + c);
        v[j][1] = *reinterpret_cast<const f32x4 *>(xr + c + 4);
        s += v[j][0][0] + v[j][0][1] + v[j][0][2] + v[j][0][3] + v[j][1][0] + v[j][1][1] + v[j][1][2] + v[j][1][3];
    }
    const float inv_c = 1.0f / (float)a.C;
    const float mu = wave_sum(s) * inv_c;
    float q = 0.f;
#pragma unroll
    for (int j = 0; j < NCH; ++j)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                v[j][h][i] -= mu;
                q = fmaf(v[j][h][i], v[j][h][i], q);
            }
    const float rstd = rsqrtf(wave_sum(q) * inv_c + a.eps);
    uint16_t *yr = static_cast<uint16_t *>(a.y) + row * a.ldy;
#pragma unroll
    for (int j = 0; j < NCH; ++j) {
        const int c = 512 * j + 8 * lane;
        f32x4 mul[2], add[2];
        if (a.scale != nullptr) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                mul[h] = *reinterpret_cast<const f32x4 *>(a.scale + c + 4 * h) + 1.0f;
                add[h] = *reinterpret_cast<const f32x4 *>(a.shift + c + 4 * h);
            }
        } else {
            const uint16_t *w = static_cast<const uint16_t *>(a.w), *b = static_cast<const uint16_t *>(a.b);
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    mul[h][i] = bf(w[c + 4 * h + i]);
                    add[h][i] = bf(b[c + 4 * h + i]);
                }
        }
        bf16x8 o;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int i = 0; i < 4; ++i) o[4 * h + i] = (__bf16)fmaf(v[j][h][i] * rstd, mul[h][i], add[h][i]);
        *reinterpret_cast<bf16x8 *>(yr + c) = o;
    }
}

template <int NCH>
__global__ __launch_bounds__(256) void rms_norm_kernel(RmsNormArgs a)
{
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= a.rows) return;
    const uint16_t *xr = static_cast<const uint16_t *>(a.x) + row * a.ldx;
    const uint16_t *w = static_cast<const uint16_t *>(a.w);
    bf16x8 v[NCH];
    float q = 0.f;
#pragma unroll
    for (int j = 0; j < NCH; ++j) {
        v[j] = *reinterpret_cast<const bf16x8 *>(xr + 512 * j + 8 * lane);
#pragma unroll
        for (int i = 0; i < 8; ++i) q = fmaf((float)v[j][i], (float)v[j][i], q);
    }
    const float r = rsqrtf(wave_sum(q) / (float)a.C + a.eps);
    uint16_t *yr = static_cast<uint16_t *>(a.y) + row * a.ldy;
#pragma unroll
    for (int j = 0; j < NCH; ++j) {
        const int c = 512 * j + 8 * lane;
        const bf16x8 wv = *reinterpret_cast<const bf16x8 *>(w + c);
        bf16x8 o;
#pragma unroll
        for (int i = 0; i < 8; ++i) o[i] = (__bf16)((float)v[j][i] * r * (float)wv[i]);
        *reinterpret_cast<bf16x8 *>(yr + c) = o;
    }
}

// adaLN vectors: one wave per output row j, lanes over the C inputs.
// Vector form (C a multiple of 8, 16-byte aligned rows and e): each wave
// takes kModRows consecutive rows; a lane walks 8-channel chunks, forms
// silu(e) of a chunk once and applies it to the chunk of every one of its
// rows (16-byte weight loads, all of a lane's issued before the first is
// used; C <= 2048).
constexpr int kModRows = 4;

__global__ __launch_bounds__(256) void modulation_vec_kernel(ModulationArgs a)
{
    constexpr int kIt = 4;  // 512-channel steps per lane: C <= 2048
    const int lane = threadIdx.x & 63;
    const int j0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * kModRows;
    if (j0 >= a.rows) return;
    const int nr = min(kModRows, a.rows - j0);
    const uint16_t *w = static_cast<const uint16_t *>(a.w) + (int64_t)j0 * a.C;
    // every weight chunk of this lane is requested before the first is used
    bf16x8 v[kIt][kModRows];
#pragma unroll
    for (int it = 0; it < kIt; ++it) {
        const int c = lane * 8 + it * 512;
#pragma unroll
        for (int r = 0; r < kModRows; ++r)
            if (c < a.C && r < nr) v[it][r] = *reinterpret_cast<const bf16x8 *>(w + (int64_t)r * a.C + c);
    }
    float s[kModRows] = {};
#pragma unroll
    for (int it = 0; it < kIt; ++it) {
        const int c = lane * 8 + it * 512;
        if (c >= a.C) break;
        const f32x4 e0 = *reinterpret_cast<const f32x4 *>(a.e + c);
        const f32x4 e1 = *reinterpret_cast<const f32x4 *>(a.e + c + 4);
        float u[8];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            u[i] = e0[i] / (1.0f + __expf(-e0[i]));
            u[4 + i] = e1[i] / (1.0f + __expf(-e1[i]));
        }
#pragma unroll
        for (int r = 0; r < kModRows; ++r) {
            if (r < nr) {
#pragma unroll
                for (int i = 0; i < 8; ++i) s[r] = fmaf((float)v[it][r][i], u[i], s[r]);
            }
        }
    }
#pragma unroll
    for (int r = 0; r < kModRows; ++r) {
        const float t = wave_sum(s[r]);
        if (lane == 0 && r < nr) a.mod[j0 + r] = t + bf(static_cast<const uint16_t *>(a.b)[j0 + r]);
    }
}

// Scalar form, any C and alignment: one wave per row.
__global__ __launch_bounds__(256) void modulation_kernel(ModulationArgs a)
{
    const int lane = threadIdx.x & 63;
    const int j = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (j >= a.rows) return;
    const uint16_t *w = static_cast<const uint16_t *>(a.w) + (int64_t)j * a.C;
    float s = 0.f;
    for (int c = lane; c < a.C; c += 64) {
        const float e = a.e[c];
        s = fmaf(bf(w[c]), e / (1.0f + __expf(-e)), s);
    }
    s = wave_sum(s);
    if (lane == 0) a.mod[j] = s + bf(static_cast<const uint16_t *>(a.b)[j]);
}

template <int BM, int EPI>
hipError_t launch_linear_t(const LinearArgs &a, hipStream_t stream)
{
    const int tiles_n = tile::tiles_along(a.N, tile::kBN), n_tiles = tile::tiles_along(a.M, BM) * tiles_n;
    hipLaunchKernelGGL((linear_kernel<BM, EPI>), dim3((unsigned)n_tiles), dim3(kThreads), 0, stream, a, tiles_n,
                       n_tiles);
    return hipGetLastError();
}

template <int BM>
hipError_t launch_linear_bm(const LinearArgs &a, hipStream_t stream)
{
    switch (a.epi) {
    case kEpiBias: return launch_linear_t<BM, kEpiBias>(a, stream);
    case kEpiBiasGelu:
        if constexpr (BM != 256) return launch_linear_t<BM, kEpiBiasGelu>(a, stream);  // see linear_plan
        break;
    case kEpiGatedRes: return launch_linear_t<BM, kEpiGatedRes>(a, stream);
    }
    return hipErrorInvalidValue;
}

template <class S, int EPI, bool WIDE>
hipError_t launch_linear4_t(const LinearArgs &a, int splits, hipStream_t stream)
{
    const int tiles_n = tile::tiles_along(a.N, S::BN), n_tiles = tile::tiles_along(a.M, S::BM) * tiles_n;
    hipLaunchKernelGGL((linear4_kernel<S, EPI, WIDE>), dim3((unsigned)n_tiles * (unsigned)splits),
                       dim3(tile::kThreads4), 0, stream, a, tiles_n, n_tiles, splits);
    return hipGetLastError();
}

template <int EPI>
hipError_t launch_reduce_t(const LinearArgs &a, int splits, hipStream_t stream)
{
    const int64_t n = (int64_t)a.M * (a.N / 8);
    hipLaunchKernelGGL(linear_reduce_kernel<EPI>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, a, splits);
    return hipGetLastError();
}

template <class S, bool WIDE = false>
hipError_t launch_linear4(const LinearArgs &a, int splits, hipStream_t stream)
{
    if constexpr (!WIDE) {
        if (splits > 1) {
            const hipError_t e = launch_linear4_t<S, tile::kPartial, false>(a, splits, stream);
            if (e != hipSuccess) return e;
            switch (a.epi) {
            case kEpiBias: return launch_reduce_t<kEpiBias>(a, splits, stream);
            case kEpiBiasGelu: return launch_reduce_t<kEpiBiasGelu>(a, splits, stream);
            case kEpiGatedRes: return launch_reduce_t<kEpiGatedRes>(a, splits, stream);
            }
            return hipErrorInvalidValue;
        }
    }
    switch (a.epi) {
    case kEpiBias: return launch_linear4_t<S, kEpiBias, WIDE>(a, 1, stream);
    case kEpiBiasGelu: return launch_linear4_t<S, kEpiBiasGelu, WIDE>(a, 1, stream);
    case kEpiGatedRes: return launch_linear4_t<S, kEpiGatedRes, WIDE>(a, 1, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace

// The tile and K split of a linear layer, by plan_tiles; the constants are
// fitted to 1002 launches (18 pairs of N and K from 256 to 14336, 19 row counts
// from 128 to 65520, three epilogues), each timed on every tile and split: the
// choice is on average 1.0 % slower than the best of them.  Measured, against
// 256 x 256 or 288 x 256 by eight waves alone:
// 1365 x 1536 x 8960 203 -> 47 us (192 x 192 in four ranges),
// 1560 x 4608 x 1536 39.7 -> 23.5 us (128 x 128), 4096 x 1536 x 8960 205 -> 94 us
// (128 x 192), 10920 x 8960 x 1536 with GELU 286 -> 254 us (256 x 256 by four
// waves); 10920 x 4608 and 10920 x 1536 stay with 288 x 256 by eight waves
// (125 and 43.7 us: 228 tiles of 288 rows are one round where 43 row blocks of
// 256 need 258 tiles), 32760 x 1536 x 1536 with the residual goes on 256 x 256
// by four waves (187 us; 288 x 256 218, 256 x 256 by eight 204).  Eight waves
// stay on 256 x 256 where K is short and the rounds are many, the epilogue much
// of a tile's time: two waves per SIMD overlap one tile's epilogue with
// another's steps (65520 x 2048 x 128 75.7 us, the best other tile 80.4;
// 32760 x 512 x 512 with the residual 34.1 against 36.0).
TilePlan linear_plan(int M, int N, int K, int epi, int n_cu, int64_t ws_bytes)
{
    if (K == 0 || K >= kWideStride) return TilePlan{kTile128x128, 1, 128, 128, 4};
    // fixed times by tile and epilogue (with the GELU, 256 x 256 by eight waves is nowhere the better one)
    static const double kFixed[8][3] = {{5.8, 9.5, 19.3}, {4.1, INFINITY, 15.6}, {7.7, 10.9, 21.6}, {4.8, 7.2, 15.5},
                                        {4.4, 6.5, 15.2}, {3.0, 6.8, 12.5},  {1.5, 2.3, 5.2},   {0.9, 1.1, 1.8}};
    const TileCost costs[] = {
        {kTile288x256, 288, 256, 8, kFixed[0][epi], 0.0, 1.222, 1.300, false},
        {kTile256x256By8, 256, 256, 8, kFixed[1][epi], 0.0, 1.113, 1.380, false},
        {kTile256x256, 256, 256, 4, kFixed[2][epi], kFixed[2][0], 0.934, 1.325, true},
        {kTile160x256, 160, 256, 4, kFixed[3][epi], kFixed[3][0], 0.737, 1.198, true},
        {kTile192x192, 192, 192, 4, kFixed[4][epi], kFixed[4][0], 0.648, 1.217, true},
        {kTile128x192, 128, 192, 4, kFixed[5][epi], kFixed[5][0], 0.497, 1.199, true},
        {kTile128x128, 128, 128, 4, kFixed[6][epi], kFixed[6][0], 0.424, 0.988, true},
        {kTile64x128, 64, 128, 4, kFixed[7][epi], kFixed[7][0], 0.396, 0.951, true},
    };
    return plan_tiles(costs, SplitCost{5.1, 8.1e6, epi == kEpiGatedRes ? 8 : 2}, M, N, K / kBK, n_cu, ws_bytes);
}

size_t linear_workspace_bytes(int M, int N, int K, int epi, int n_cu)
{
    if (M == 0 || N == 0 || K == 0) return 0;
    const TilePlan p = linear_plan(M, N, K, epi, n_cu, INT64_MAX);
    return p.splits > 1 ? (size_t)p.splits * M * N * sizeof(float) : 0;
}

hipError_t launch_linear(const LinearArgs &a, hipStream_t stream)
{
    if (a.M == 0 || a.N == 0) return hipSuccess;
    // no steps at all, or strides for which the offsets within a tile may leave 32 bits
    if (a.K == 0 || a.lda >= kWideStride || a.K >= kWideStride) return launch_linear4<Tile128x128, true>(a, 1, stream);
    const TilePlan p = linear_plan(a.M, a.N, a.K, a.epi, device_cu_count(), a.ws != nullptr ? a.ws_bytes : 0);
    switch (p.tile) {
    case kTile256x256: return launch_linear4<Tile256x256>(a, p.splits, stream);
    case kTile160x256: return launch_linear4<Tile160x256>(a, p.splits, stream);
    case kTile192x192: return launch_linear4<Tile192x192>(a, p.splits, stream);
    case kTile128x128: return launch_linear4<Tile128x128>(a, p.splits, stream);
    case kTile128x192: return launch_linear4<Tile128x192>(a, p.splits, stream);
    case kTile64x128: return launch_linear4<Tile64x128>(a, p.splits, stream);
    case kTile288x256: return launch_linear_bm<288>(a, stream);
    case kTile256x256By8: return launch_linear_bm<256>(a, stream);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_layer_norm(const LayerNormArgs &a, hipStream_t stream)
{
    const dim3 grid((unsigned)((a.rows + 3) / 4)), block(256);
    switch (a.C / 512) {
    case 1: hipLaunchKernelGGL(layer_norm_kernel<1>, grid, block, 0, stream, a); break;
    case 2: hipLaunchKernelGGL(layer_norm_kernel<2>, grid, block, 0, stream, a); break;
    case 3: hipLaunchKernelGGL(layer_norm_kernel<3>, grid, block, 0, stream, a); break;
    case 4: hipLaunchKernelGGL(layer_norm_kernel<4>, grid, block, 0, stream, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_rms_norm(const RmsNormArgs &a, hipStream_t stream)
{
    const dim3 grid((unsigned)((a.rows + 3) / 4)), block(256);
    switch (a.C / 512) {
    case 1: hipLaunchKernelGGL(rms_norm_kernel<1>, grid, block, 0, stream, a); break;
    case 2: hipLaunchKernelGGL(rms_norm_kernel<2>, grid, block, 0, stream, a); break;
    case 3: hipLaunchKernelGGL(rms_norm_kernel<3>, grid, block, 0, stream, a); break;
    case 4: hipLaunchKernelGGL(rms_norm_kernel<4>, grid, block, 0, stream, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_modulation(const ModulationArgs &a, hipStream_t stream)
{
    const bool vec = a.C % 8 == 0 && a.C <= 2048 && ((uintptr_t)a.w & 15) == 0 && ((uintptr_t)a.e & 15) == 0;
    if (vec) {
        const int per_block = 4 * kModRows;
        hipLaunchKernelGGL(modulation_vec_kernel, dim3((unsigned)((a.rows + per_block - 1) / per_block)), dim3(256), 0,
                           stream, a);
    } else {
        hipLaunchKernelGGL(modulation_kernel, dim3((unsigned)((a.rows + 3) / 4)), dim3(256), 0, stream, a);
    }
    return hipGetLastError();
}

}  // namespace regenvc
