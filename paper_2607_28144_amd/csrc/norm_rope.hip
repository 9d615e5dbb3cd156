// gfx950 q/k RMSNorm + 3D rotary position embedding: the steps between the
// QKV projection and self-attention in a block of the video diffusion
// transformer, producing the attention kernels' bf16 [B, S, H, D] inputs.
//
// Per token: r = 1/sqrt(mean of the squares of its H*D channels + eps),
// y = x * r * w, then per head a rotation of each (2i, 2i+1) pair by
// pos_a * theta^(-2k/d_a), with pairs split over the frame, row and column
// axes of the latent grid (22/21/21 pairs at D = 128).
//
// HBM-bound: a token's q and k are read once and written once.  One wave
// handles a few tokens, q and k together (they share the rotation angles):
// each lane keeps its 16-byte chunks of both in registers between the sum of
// squares (wave reduction) and the scaled, rotated write-back, and requests
// those of its next token before it works on this one.  A lane's chunks lie
// 512 channels apart, a whole number of heads: they rotate by the same angles,
// whose frequencies are formed once per wave and sines and cosines once per
// token.  10920 tokens of 12 heads x 128 (134 MB): 34.9 -> 25.0 us (5.3 TB/s;
// a large copy reaches 5.1), 1560 tokens 8.9 -> 6.2 us, 300 tokens 6.2 -> 4.5
// us; with the angles formed per chunk and 64-bit divisions per token the
// vector unit was what bound it.  What a wave holds costs it neighbours: 188
// registers at 1536 channels are two waves per SIMD, so the window's 3640 waves
// run as 1.8 rounds of 2048; from 4097 to 8192 channels (256 registers, no next
// token held) one wave per SIMD still takes less time than two of the former
// kernel did (10920 tokens of 40 heads x 128 138 -> 102 us, of 64 heads 215 ->
// 154 us).
#include "attn_kernels.hpp"

#include <math.h>

namespace regenvc {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));  // eight bf16, the first of a pair in the low half
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// Waves launched per compute unit, at most: where registers allow fewer at a
// time, the rest follow.
constexpr int kWavesPerCu = 16;
constexpr float kInv2Pi = 0.15915494309189535f;

// the two bf16 of a pair, and a pair rounded to nearest even
__device__ __forceinline__ float lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float hi(uint32_t u) { return __uint_as_float(u & 0xffff0000u); }
__device__ __forceinline__ uint32_t pack(float a, float b)
{
    const bf16x2 v = {(__bf16)a, (__bf16)b};
    return __builtin_bit_cast(uint32_t, v);
}

__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
    return v;
}

// NCH: 16-byte chunks per lane and tensor (C = H D <= 512 NCH).  Wave w handles
// tokens w, w + waves, ...
template <int D, int NCH>
__global__ __launch_bounds__(64) void qk_norm_rope_kernel(NormRopeArgs a)
{
    const int lane = threadIdx.x & 63;
    const int64_t tokens = (int64_t)a.B * a.S;
    const int C = a.H * D, nchunk = C / 8;
    constexpr int P = D / 2, ph = D / 6, pf = P - 2 * ph;  // pairs of a head, of its row and column axes, of its frame axis

    // this lane's place in its heads, and the frequencies (radians per position) and axes of its four pairs
    const int d0 = (lane * 8) % D, h0 = (lane * 8) / D;
    constexpr int kHeadStep = 512 / D;
    float freq[4];
    int axis[4];
#pragma unroll
    for (int pp = 0; pp < 4; ++pp) {
        const int i = d0 / 2 + pp;  // pair index within the head
        axis[pp] = i < pf ? 0 : i < pf + ph ? 1 : 2;
        const int kk = i - (i < pf ? 0 : i < pf + ph ? pf : pf + ph), pairs = i < pf ? pf : ph;
        freq[pp] = exp2f(-(float)kk / (float)pairs * a.log2_theta);
    }
    // with up to four chunks per lane, the weights and the next token's chunks are held as well
    constexpr bool KEEP = NCH <= 4;
    auto weight = [&](const void *w, int j) {
        return *reinterpret_cast<const u32x4 *>(static_cast<const uint16_t *>(w) + (lane + 64 * j) * 8);
    };
    u32x4 wq[KEEP ? NCH : 1], wk[KEEP ? NCH : 1];
    if constexpr (KEEP) {
#pragma unroll
        for (int j = 0; j < NCH; ++j)
            if (lane + 64 * j < nchunk) wq[j] = weight(a.w_q, j), wk[j] = weight(a.w_k, j);
    }
    auto place = [&](int64_t token, int64_t &b, int64_t &t) {
        b = a.B > 1 ? token / a.S : 0;
        t = token - b * a.S;
    };
    auto load = [&](int64_t token, u32x4 (&qx)[NCH], u32x4 (&kx)[NCH]) {
        int64_t b, t;
        place(token, b, t);
        const uint16_t *qi = static_cast<const uint16_t *>(a.q_in) + b * a.qi_sb + t * a.qi_ss + d0;
        const uint16_t *ki = static_cast<const uint16_t *>(a.k_in) + b * a.ki_sb + t * a.ki_ss + d0;
#pragma unroll
        for (int j = 0; j < NCH; ++j)
            if (lane + 64 * j < nchunk) {
                const int h = h0 + kHeadStep * j;
                qx[j] = *reinterpret_cast<const u32x4 *>(qi + h * a.qi_sh);
                kx[j] = *reinterpret_cast<const u32x4 *>(ki + h * a.ki_sh);
            }
    };
    u32x4 qv[NCH], kv[NCH];
    int64_t token = blockIdx.x;
    if (token < tokens) load(token, qv, kv);
    for (; token < tokens; token += gridDim.x) {
        float sq = 0.f, sk = 0.f;
#pragma unroll
        for (int j = 0; j < NCH; ++j) {
            if (lane + 64 * j < nchunk) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    sq = fmaf(hi(qv[j][e]), hi(qv[j][e]), fmaf(lo(qv[j][e]), lo(qv[j][e]), sq));
                    sk = fmaf(hi(kv[j][e]), hi(kv[j][e]), fmaf(lo(kv[j][e]), lo(kv[j][e]), sk));
                }
            }
        }
        u32x4 qn[KEEP ? NCH : 1], kn[KEEP ? NCH : 1];
        if constexpr (KEEP) {
            if (token + gridDim.x < tokens) load(token + gridDim.x, qn, kn);
        }
        // 1/sqrt of q's mean square in the lower lanes and k's in the upper: one
        // sequence for both.  The mean by division: a product with 1 / C is
        // rounded twice.
        const float tq = wave_sum(sq), tk = wave_sum(sk);
        const int r = __float_as_int(1.0f / sqrtf((lane < 32 ? tq : tk) / (float)C + a.eps));
        const float rq = __int_as_float(__builtin_amdgcn_readlane(r, 0));
        const float rk = __int_as_float(__builtin_amdgcn_readlane(r, 32));

        // this token's grid position (token0 + S < 2^32) and its sines and cosines
        int64_t b, t;
        place(token, b, t);
        const uint32_t g = (uint32_t)a.token0 + (uint32_t)t, row = g / (uint32_t)a.grid_w;
        const uint32_t frame = row / (uint32_t)a.grid_h;
        const float pos[3] = {(float)frame, (float)(row - frame * (uint32_t)a.grid_h),
                              (float)(g - row * (uint32_t)a.grid_w)};
        float sn[4], cs[4];
#pragma unroll
        for (int pp = 0; pp < 4; ++pp) {
            // angle pos_a * theta^(-2k/d_a), d_a = 2 * pairs, in turns; the
            // hardware sine/cosine take turns, reduced to [0, 1) first (exact)
            const float p = axis[pp] == 0 ? pos[0] : axis[pp] == 1 ? pos[1] : pos[2];
            const float turns = __builtin_amdgcn_fractf(p * freq[pp] * kInv2Pi);
            sn[pp] = __builtin_amdgcn_sinf(turns), cs[pp] = __builtin_amdgcn_cosf(turns);
        }
        uint16_t *qo = static_cast<uint16_t *>(a.q_out) + b * a.qo_sb + t * a.qo_ss + d0;
        uint16_t *ko = static_cast<uint16_t *>(a.k_out) + b * a.ko_sb + t * a.ko_ss + d0;
#pragma unroll
        for (int j = 0; j < NCH; ++j) {
            if (lane + 64 * j >= nchunk) continue;
            const int h = h0 + kHeadStep * j;
            const u32x4 wqj = KEEP ? wq[KEEP ? j : 0] : weight(a.w_q, j), wkj = KEEP ? wk[KEEP ? j : 0] : weight(a.w_k, j);
            u32x4 oq, ok;
#pragma unroll
            for (int pp = 0; pp < 4; ++pp) {
                const float q0 = lo(qv[j][pp]) * rq * lo(wqj[pp]), q1 = hi(qv[j][pp]) * rq * hi(wqj[pp]);
                const float k0 = lo(kv[j][pp]) * rk * lo(wkj[pp]), k1 = hi(kv[j][pp]) * rk * hi(wkj[pp]);
                oq[pp] = pack(q0 * cs[pp] - q1 * sn[pp], q0 * sn[pp] + q1 * cs[pp]);
                ok[pp] = pack(k0 * cs[pp] - k1 * sn[pp], k0 * sn[pp] + k1 * cs[pp]);
            }
            *reinterpret_cast<u32x4 *>(qo + h * a.qo_sh) = oq;
            *reinterpret_cast<u32x4 *>(ko + h * a.ko_sh) = ok;
        }
        if constexpr (KEEP) {
#pragma unroll
            for (int j = 0; j < NCH; ++j) qv[j] = qn[j], kv[j] = kn[j];
        } else {
            break;  // one token per wave
        }
    }
}

template <int D>
hipError_t launch_d(const NormRopeArgs &a, hipStream_t stream)
{
    // each wave has its share of the tokens; one of more than four chunks per
    // lane has no registers for a next token
    const int64_t tokens = (int64_t)a.B * a.S, slots = (int64_t)device_cu_count() * kWavesPerCu;
    const int nch = (a.H * D + 511) / 512;
    const int64_t per = nch <= 4 ? (tokens + slots - 1) / slots : 1;
    const dim3 grid((unsigned)((tokens + per - 1) / per)), block(64);
    switch (nch) {
    case 1: hipLaunchKernelGGL((qk_norm_rope_kernel<D, 1>), grid, block, 0, stream, a); break;
    case 2: hipLaunchKernelGGL((qk_norm_rope_kernel<D, 2>), grid, block, 0, stream, a); break;
    case 3: hipLaunchKernelGGL((qk_norm_rope_kernel<D, 3>), grid, block, 0, stream, a); break;
    case 4: hipLaunchKernelGGL((qk_norm_rope_kernel<D, 4>), grid, block, 0, stream, a); break;
    default:
        if (nch > 16) return hipErrorInvalidValue;
        if (nch <= 8)
            hipLaunchKernelGGL((qk_norm_rope_kernel<D, 8>), grid, block, 0, stream, a);
        else
            hipLaunchKernelGGL((qk_norm_rope_kernel<D, 16>), grid, block, 0, stream, a);
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_norm_rope(const NormRopeArgs &a, hipStream_t stream)
{
    return a.D == 128 ? launch_d<128>(a, stream) : launch_d<64>(a, stream);
}

}  // namespace regenvc
