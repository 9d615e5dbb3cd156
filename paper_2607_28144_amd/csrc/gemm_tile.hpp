// The bf16 MFMA tile kernels of the linear layers of the diffusion block
// (dense rows) and of the VAE's causal 3D convolution (rows gathered as an
// implicit GEMM): out[m][n] = epilogue(sum_k A[m][k] W[n][k]).  Four waves per
// tile (mma4, store4) for most shapes; eight (tile_body) for tiles of 288 rows
// and for some of 256.
//
// Eight waves (dense rows only).  Workgroup = 8 waves (two per SIMD) = one BM
// x 256 output tile; the waves form a 2 x 4 grid, each owning BM / 2 rows x 64
// channels on v_mfma_f32_16x16x32_bf16.  The product is formed transposed, C^T
// = W A^T, so that a lane's accumulator holds four consecutive output channels
// of one row (what the epilogues want).  K advances in steps of 64: both
// operand tiles go HBM -> LDS with global_load_lds_dwordx4 (no register
// staging) into a double-buffered LDS ring; rows are 128 bytes, 16-byte chunk c
// of row r stored at chunk c ^ ((r >> 1) & 7), which makes the fragment reads
// (16 rows, one chunk) bank-conflict free.  Tiles are dealt XCD-aware: each XCD
// takes a contiguous range of tiles, numbered in groups of four row blocks
// swept across the channel blocks, so that the tiles resident on an XCD share
// their operand blocks through its L2.
//
// Four waves: see below.  Their operand rows are a policy that gives, for each
// of a lane's copy rows, the address of the 16 bytes to copy at K step kt: a
// dense row, or a tap of a convolution patch, or a page of zeros for padding.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace regenvc {
namespace tile {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) bf16x8 lds_bf16x8;
typedef __attribute__((address_space(3))) char lds_char;

constexpr int kWaves = 8;
constexpr int kThreads = 64 * kWaves;
constexpr int kBK = 64;               // K per step (two 32-deep MFMA steps)
constexpr int kRowBytes = kBK * 2;
constexpr int kGroupM = 4;            // row blocks per group of the tile order

enum Epi : int32_t {
    kBias = 0,        // out bf16 = y + bias
    kBiasGelu = 1,    // out bf16 = gelu_tanh(y + bias)
    kGatedRes = 2,    // out f32 (in place) = out + gate[n] * (y + bias[n])   (gate may be null: 1)
    kBiasSilu = 3,    // out bf16 = silu(y + bias)
    kPartial = 4,     // out f32 = y over this workgroup's share of K (split-K partial, no bias)
};

// Output side of a tile launch.
struct Out {
    const uint16_t *bias; // [N] bf16 or null
    const float *gate;    // [N] f32 or null (kGatedRes)
    void *out;            // bf16 or f32 [M, N], row stride ldo
    int64_t ldo;
    int32_t M, N;
};

#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
// 16-byte HBM -> LDS copy (global_load_lds_dwordx4): lane i's 16 bytes land
// at lds_base + 16 * i.  Inline asm so that the compiler does not order it
// against the LDS reads of the other ring stage; completion is awaited with
// an explicit s_waitcnt vmcnt before the barrier that publishes the stage.
__device__ __forceinline__ void lds_copy16(const void *gptr, uint32_t lds_base)
{
    const uint32_t base = __builtin_amdgcn_readfirstlane(lds_base);  // wave-uniform by construction
    __asm__ volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(base), "v"(gptr) : "m0");
}
#pragma clang diagnostic pop

__device__ __forceinline__ void wait_all_copies()
{
    __asm__ volatile("s_waitcnt vmcnt(0)" : : : "memory");
}

__device__ __forceinline__ int swz(int row, int chunk)
{
    return chunk ^ ((row >> 1) & 7);
}

// Activations of the epilogues, in the sigmoid form with the hardware
// base-2 exponential and reciprocal (both within an ulp or two of fp32,
// far below the bf16 rounding that follows): no fp32 division.
//   gelu_tanh(x) = x/2 (1 + tanh(u)) = x sigmoid(2u),  u = sqrt(2/pi) (x + 0.044715 x^3),
//   sigmoid(2u) = 1 / (1 + 2^z),  z = -2 log2(e) u = x (kG1 + kG3 x^2).
__device__ __forceinline__ float gelu_tanh(float x)
{
    constexpr float kG1 = -2.0f * 1.4426950408889634f * 0.7978845608028654f;
    constexpr float kG3 = kG1 * 0.044715f;
    const float z = x * fmaf(kG3, x * x, kG1);
    return x * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(z));
}

// silu(x) = x sigmoid(x) = x / (1 + 2^(-x log2 e)).
__device__ __forceinline__ float silu(float x)
{
    return x * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * x));
}

__device__ __forceinline__ float bf(uint16_t b)
{
    return __uint_as_float(((uint32_t)b) << 16);
}

// Tile (row block, channel block) of workgroup bid among n_tiles, XCD-aware:
// workgroup i runs on XCD i % 8; XCD x takes a contiguous range of tiles.
// Tiles are numbered in groups of kGroupM row blocks swept across the channel
// blocks (row block fastest), so the ~32 tiles resident on an XCD at a time
// cover about 4 row blocks x 8 channel blocks: each A row block and W block
// they read serves several of them from the XCD's L2.
__device__ __forceinline__ void tile_of(int bid, int tiles_n, int n_tiles, int &tm, int &tn)
{
    const int xcd = bid & 7, slot = bid >> 3;
    const int tile = xcd * (n_tiles >> 3) + min(xcd, n_tiles & 7) + slot;
    const int tiles_m = n_tiles / tiles_n;
    const int group = tile / (kGroupM * tiles_n), in_group = tile - group * kGroupM * tiles_n;
    const int gm = min(tiles_m - group * kGroupM, kGroupM);
    tm = group * kGroupM + in_group % gm;
    tn = in_group / gm;
}

// One BM x BN output tile of eight waves: rows a [M, K] (row stride lda), w [N, K].
constexpr int kBN = 256;
template <int BM, int EPI>
__device__ __forceinline__ void tile_body(const uint16_t *a, int64_t lda, const uint16_t *w, int K, const Out &o,
                                          int tiles_n, int n_tiles, char *smem)
{
    constexpr int WN = 4, NB = 4;        // waves across, 16-channel MFMA blocks of each
    constexpr int BN = kBN;
    constexpr int WM = BM / 2;           // rows per wave
    constexpr int MB = WM / 16;          // 16-row MFMA blocks per wave
    constexpr int A_BYTES = BM * kRowBytes;
    constexpr int W_BYTES = BN * kRowBytes;
    constexpr int STAGE = A_BYTES + W_BYTES;
    constexpr int A_INSTR = A_BYTES / 1024;  // 1 KB (8 rows) per wave copy instruction
    constexpr int W_INSTR = W_BYTES / 1024;
    constexpr int A_PER = (A_INSTR + kWaves - 1) / kWaves;
    constexpr int W_PER = W_INSTR / kWaves;
    static_assert(WM % 16 == 0 && BN == 16 * NB * WN && W_INSTR % kWaves == 0, "tile shape");

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int g = lane >> 4, x = lane & 15;

    int tm, tn;
    tile_of((int)blockIdx.x, tiles_n, n_tiles, tm, tn);
    const int m0 = tm * BM, n0 = tn * BN;

    // this lane's copies: instruction j of a tile covers its rows 8j..8j+7;
    // lane l fills LDS chunk l % 8 of row 8j + l / 8, which holds global
    // chunk swz(row, l % 8).  Rows past the end re-read the last row (never
    // stored).
    const uint16_t *asrc[A_PER];
#pragma unroll
    for (int i = 0; i < A_PER; ++i) {
        const int j = min(wave + i * kWaves, A_INSTR - 1);
        const int r = j * 8 + (lane >> 3);
        asrc[i] = a + (int64_t)min(m0 + r, o.M - 1) * lda + swz(r, lane & 7) * 8;
    }
    const uint16_t *wsrc[W_PER];
#pragma unroll
    for (int i = 0; i < W_PER; ++i) {
        const int r = (wave + i * kWaves) * 8 + (lane >> 3);
        const int gr = min(n0 + r, o.N - 1);
        wsrc[i] = w + (int64_t)gr * K + swz(r, lane & 7) * 8;
    }
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char *)smem;
    auto issue = [&](int kt, int st) {
        const uint32_t sa = lds0 + st * STAGE, sw = sa + A_BYTES;
#pragma unroll
        for (int i = 0; i < A_PER; ++i) {
            const int j = wave + i * kWaves;
            if (j < A_INSTR) lds_copy16(asrc[i] + kt * kBK, sa + j * 1024);
        }
#pragma unroll
        for (int i = 0; i < W_PER; ++i) lds_copy16(wsrc[i] + kt * kBK, sw + (wave + i * kWaves) * 1024);
    };

    f32x4 acc[NB][MB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) acc[nb][mb] = f32x4{0.f, 0.f, 0.f, 0.f};

    const int nk = K / kBK;
    issue(0, 0);
    for (int kt = 0; kt < nk; ++kt) {
        const int st = kt & 1;
        wait_all_copies();   // this wave's copies of step kt landed
        __syncthreads();     // ... and every wave's; step kt-1's stage is free
        if (kt + 1 < nk) issue(kt + 1, st ^ 1);
        const lds_char *sa = (const lds_char *)smem + st * STAGE;
        const lds_char *sw = sa + A_BYTES;
        // the step's 2 x MB groups of 4 MFMAs (k half ks, row block mb),
        // each A fragment read two groups ahead of its MFMAs (a ring of 3)
        // and the second k half's W fragments read at the start, the order
        // pinned so that the LDS latency passes under earlier MFMAs
        auto afrag = [&](int s) {
            const int r = wm * WM + (s % MB) * 16 + x;
            return *(const lds_bf16x8 *)(sa + r * kRowBytes + swz(r, (s / MB) * 4 + g) * 16);
        };
        auto wfrag = [&](int ks, int nb) {
            const int r = wn * (16 * NB) + nb * 16 + x;
            return *(const lds_bf16x8 *)(sw + r * kRowBytes + swz(r, ks * 4 + g) * 16);
        };
        bf16x8 wf[2][NB], ar[3];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) wf[0][nb] = wfrag(0, nb);
        ar[0] = afrag(0);
        ar[1] = afrag(1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < 2 * MB; ++s) {
            if (s + 2 < 2 * MB) ar[(s + 2) % 3] = afrag(s + 2);
            if (s == 0) {
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) wf[1][nb] = wfrag(1, nb);
            }
            const int ks = s / MB, mb = s % MB;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
                acc[nb][mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[ks][nb], ar[s % 3], acc[nb][mb], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    }

    // epilogue: acc[nb][mb][i] = y[m0 + wm*WM + mb*16 + x][n0 + wn*16*NB + nb*16 + 4g + i]
    constexpr bool BF16_OUT = EPI == kBias || EPI == kBiasGelu;
    if constexpr (BF16_OUT) {
        // A whole-width tile with 16-byte aligned rows goes out as full rows:
        // the values are staged in the (now idle) LDS, row-major with 16-byte
        // chunk c of row r at chunk c ^ (r & 15), and each store instruction
        // then writes whole 16-byte chunks of consecutive rows instead of 8
        // bytes of each of 16 rows.
        if (n0 + BN <= o.N && (reinterpret_cast<uintptr_t>(o.out) & 15) == 0 && (o.ldo & 7) == 0) {
            constexpr int CH = BN / 8;  // 16-byte chunks per staged row
            static_assert(CH % 16 == 0 && (BM * CH) % kThreads == 0, "staging shape");
            __syncthreads();  // every wave is done reading the ring
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const int n = n0 + wn * (16 * NB) + nb * 16 + 4 * g;
                f32x4 bv = {0.f, 0.f, 0.f, 0.f};
                if (o.bias != nullptr) {
                    const uint64_t b4 = *reinterpret_cast<const uint64_t *>(o.bias + n);
#pragma unroll
                    for (int i = 0; i < 4; ++i) bv[i] = bf((uint16_t)(b4 >> (16 * i)));
                }
                const int c = wn * 2 * NB + nb * 2 + g / 2;
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) {
                    const int r = wm * WM + mb * 16 + x;
                    const f32x4 y = acc[nb][mb] + bv;
                    bf16x4 w;
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        w[i] = (__bf16)(EPI == kBiasGelu ? gelu_tanh(y[i]) : y[i]);
                    *(__attribute__((address_space(3))) bf16x4 *)((lds_char *)smem + r * (BN * 2) +
                                                                 ((c ^ (r & 15)) * 16) + (g & 1) * 8) = w;
                }
            }
            __syncthreads();
#pragma unroll
            for (int it = 0; it < BM * CH / kThreads; ++it) {
                const int id = it * kThreads + (int)threadIdx.x;
                const int r = id / CH, c = id % CH;
                const bf16x8 v = *(const lds_bf16x8 *)((const lds_char *)smem + r * (BN * 2) + ((c ^ (r & 15)) * 16));
                if (m0 + r < o.M)
                    *reinterpret_cast<bf16x8 *>(static_cast<uint16_t *>(o.out) + (int64_t)(m0 + r) * o.ldo + n0 +
                                                c * 8) = v;
            }
            return;
        }
    }
    if constexpr (EPI == kGatedRes) {
        // The same for the read-modify-write of the fp32 residual, in two
        // passes over half the tile's channels each (the staged fp32 half
        // tile fits the LDS): y + bias is staged, and the lane that owns a
        // 16-byte chunk of a row adds gate * y to it with whole-chunk loads
        // and stores of consecutive rows.
        if (n0 + BN <= o.N && (reinterpret_cast<uintptr_t>(o.out) & 15) == 0 && (o.ldo & 3) == 0) {
            constexpr int HALF = BN / 2;  // channels per pass
            constexpr int CH = HALF / 4;  // 16-byte chunks per staged row
            constexpr int WCH = 16 * NB;  // channels of one wave column
            static_assert(HALF % WCH == 0 && CH % 16 == 0 && (BM * CH) % kThreads == 0, "staging shape");
#pragma unroll
            for (int pass = 0; pass < 2; ++pass) {
                __syncthreads();  // the ring (first pass) or the previous half is no longer read
                if (wn * WCH / HALF == pass) {
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) {
                        const int col = wn * WCH + nb * 16 + 4 * g;  // channel within the tile
                        f32x4 bv = {0.f, 0.f, 0.f, 0.f};
                        if (o.bias != nullptr) {
                            const uint64_t b4 = *reinterpret_cast<const uint64_t *>(o.bias + n0 + col);
#pragma unroll
                            for (int i = 0; i < 4; ++i) bv[i] = bf((uint16_t)(b4 >> (16 * i)));
                        }
                        const int c = (col - pass * HALF) / 4;
#pragma unroll
                        for (int mb = 0; mb < MB; ++mb) {
                            const int r = wm * WM + mb * 16 + x;
                            *(__attribute__((address_space(3))) f32x4 *)((lds_char *)smem + r * (HALF * 4) +
                                                                        ((c ^ (r & 15)) * 16)) = acc[nb][mb] + bv;
                        }
                    }
                }
                __syncthreads();
#pragma unroll 2
                for (int it = 0; it < BM * CH / kThreads; ++it) {
                    const int id = it * kThreads + (int)threadIdx.x;
                    const int r = id / CH, c = id % CH;
                    if (m0 + r >= o.M) continue;
                    const int n = n0 + pass * HALF + c * 4;
                    const f32x4 y =
                        *(const __attribute__((address_space(3))) f32x4 *)((const lds_char *)smem + r * (HALF * 4) +
                                                                         ((c ^ (r & 15)) * 16));
                    const f32x4 gv = o.gate != nullptr ? *reinterpret_cast<const f32x4 *>(o.gate + n)
                                                       : f32x4{1.f, 1.f, 1.f, 1.f};
                    f32x4 *p = reinterpret_cast<f32x4 *>(static_cast<float *>(o.out) + (int64_t)(m0 + r) * o.ldo + n);
                    *p = *p + gv * y;
                }
            }
            return;
        }
    }
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const int n = n0 + wn * (16 * NB) + nb * 16 + 4 * g;
        if (n >= o.N) continue;
        f32x4 bv = {0.f, 0.f, 0.f, 0.f};
        if (o.bias != nullptr) {
            const uint64_t b4 = *reinterpret_cast<const uint64_t *>(o.bias + n);
#pragma unroll
            for (int i = 0; i < 4; ++i) bv[i] = bf((uint16_t)(b4 >> (16 * i)));
        }
        f32x4 gv = {1.f, 1.f, 1.f, 1.f};
        if (EPI == kGatedRes && o.gate != nullptr) gv = *reinterpret_cast<const f32x4 *>(o.gate + n);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            const int m = m0 + wm * WM + mb * 16 + x;
            if (m >= o.M) continue;
            const f32x4 y = acc[nb][mb] + bv;
            if constexpr (EPI == kGatedRes) {
                f32x4 *p = reinterpret_cast<f32x4 *>(static_cast<float *>(o.out) + (int64_t)m * o.ldo + n);
                *p = *p + gv * y;
            } else {
                bf16x4 w;
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    w[i] = (__bf16)(EPI == kBiasGelu ? gelu_tanh(y[i]) : y[i]);
                *reinterpret_cast<bf16x4 *>(static_cast<uint16_t *>(o.out) + (int64_t)m * o.ldo + n) = w;
            }
        }
    }
}

// LDS bytes of a BM x 256 tile of eight waves: its double-buffered ring, or the
// output staging if that is larger.
template <int BM>
constexpr int lds_bytes()
{
    constexpr int ring = 2 * (BM + kBN) * kRowBytes;
    constexpr int staging = BM * kBN * 2;  // bf16 tile, or half of it in fp32
    return ring > staging ? ring : staging;
}

// ---------------------------------------------------------------- four waves
// The same product by four waves, one (or, for small tiles, two or three
// workgroups') per SIMD, each owning (16 MB) rows x (16 NB) channels of a
// (32 MB) x (32 NB) tile.
//
// What bounds it and why this form.  One 64-deep K step is 2 MB NB MFMAs of
// 16-17 cycles per wave; beside them the LDS takes the step's copies at 64
// bytes a cycle and serves the fragment reads at 128.  256 x 256: 2176 cycles
// of MFMA against 2048 of LDS; 192 x 192: 1224 against 1536 (measured: 1474 a
// step); 128 x 128: 544 against 1024 (1075).  The eight-wave tile (144 x 64
// per wave) reads half as much again per MFMA: 2752 against 2304 (3228).
// Both halves of a step (32 deep each) have their fragments
// in registers before their MFMAs begin: the reads of a step's second half
// run beside the MFMAs of its first, those of the next step's first half
// beside the MFMAs of its second, so that nothing waits for LDS after the
// step's one barrier.  A wave has its SIMD to itself: every cycle in which it
// cannot issue is a cycle without MFMAs.  The loop therefore has no branch at
// all (the copies of the last two steps read the last step's data again,
// into stages nobody reads) and no vector address arithmetic (32-bit lane
// offsets, scalar bases), and its copies are spread one per eight MFMAs: A's
// over the first half, into a ring of three stages, W's over the second,
// into a ring of two.  Measured on 36 workgroups of 256 x 256 x 8960: 137 us;
// with a branch around the copies 174 us, one around each copy 248 us,
// without any copies 135 us.  8192 x 8192 x 8192: 724 us (1520 TFLOP/s), the
// eight-wave tile kernel 782-792 us.
template <int MB_, int NB_, int AS_, int WPE_>
struct Shape4 {
    static constexpr int MB = MB_, NB = NB_;  // 16-row and 16-channel blocks per wave
    static constexpr int AS = AS_;            // stages of the A ring (W's has two)
    static constexpr int WPE = WPE_;          // waves per SIMD: workgroups per compute unit
    static constexpr int BM = 32 * MB, BN = 32 * NB;
    static constexpr int A_BYTES = BM * kRowBytes, W_BYTES = BN * kRowBytes;
    static constexpr int LDS = AS * A_BYTES + 2 * W_BYTES;
    static_assert(MB * NB <= 64 && (MB * NB) % 2 == 0 && (AS == 2 || AS == 3), "tile shape");
    static_assert(LDS * WPE <= 160 * 1024, "the workgroups of one compute unit fit its LDS");
};

constexpr int kThreads4 = 256;

#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
// 16-byte HBM -> LDS copies, lane i to lds_base + 16 i (a wave-uniform
// address): with a scalar base and a 32-bit lane offset, and with a 64-bit
// lane address.  One wait state between the write of M0 and its use.
__device__ __forceinline__ void lds_copy16_s(const void *base, uint32_t off, uint32_t lds_base)
{
    __asm__ volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                     :
                     : "s"(lds_base), "v"(off), "s"(base)
                     : "m0");
}
__device__ __forceinline__ void lds_copy16_v(const void *ptr, uint32_t lds_base)
{
    __asm__ volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                     :
                     : "s"(lds_base), "v"(ptr)
                     : "m0");
}
#pragma clang diagnostic pop

// Rows of a [rows, K] bf16 matrix (row stride ld elements) as a copy source:
// copies read row r (clamped to the last one; those rows are never stored),
// 16-byte chunk c, K step kt.  WIDE: strides for which the offsets within a
// tile do not fit 32 bits.
template <bool WIDE>
struct Dense {
    const uint16_t *p;
    int64_t ld;
    int rows;
    int r0;
    struct Row {
        const char *ptr;
        uint32_t off;
    };
    __device__ Row row(int r, int chunk) const
    {
        Row q;
        const int64_t m = min(r0 + r, rows - 1);
        if constexpr (WIDE) {
            q.ptr = reinterpret_cast<const char *>(p + m * ld) + chunk * 16;
            q.off = 0;
        } else {
            q.ptr = nullptr;
            q.off = (uint32_t)(m - r0) * (uint32_t)ld * 2 + chunk * 16;
        }
        return q;
    }
    // what the copies of K step kt share (wave-uniform)
    struct Step {
        const char *base;
    };
    __device__ Step at(int kt) const
    {
        const int64_t k = (int64_t)kt * kRowBytes;
        if constexpr (WIDE)
            return Step{reinterpret_cast<const char *>(k)};
        else
            return Step{reinterpret_cast<const char *>(p + (int64_t)r0 * ld) + k};
    }
    // a row's copy at a step: its address (vector work, done a few MFMAs ahead), and the copy
    struct Addr {
        const char *ptr;
        uint32_t off;
    };
    __device__ Addr addr(const Row &q, const Step &s) const
    {
        if constexpr (WIDE)
            return Addr{q.ptr + reinterpret_cast<int64_t>(s.base), 0};
        else
            return Addr{s.base, q.off};
    }
    __device__ void copy(const Addr &a, uint32_t lds) const
    {
        if constexpr (WIDE)
            lds_copy16_v(a.ptr, lds);
        else
            lds_copy16_s(a.ptr, a.off, lds);
    }
};

// c += a b.  Tiles with one wave per SIMD keep up to 256 accumulation
// registers: written as an instruction whose result is tied to its addend,
// since the allocator otherwise renames the accumulators and moves them back
// on every K step (116 to 608 register moves per step of 128 MFMAs).  The
// compiler inserts no wait states around it: its operands come from LDS
// reads (counted), and mma4 ends with the wait states that a vector read of
// the accumulators needs.
template <class S>
__device__ __forceinline__ void mfma_into(f32x4 &c, bf16x8 a, bf16x8 b)
{
    if constexpr (S::WPE == 1)
        __asm__("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
    else
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// The K loop over steps [k0, k1) (k1 > k0): acc[nb][mb][i] = the sum for row
// 16 MB wm + 16 mb + x and channel 16 NB wn + 16 nb + 4 g + i of the tile,
// lane = 16 g + x.  On return no copy is in flight.
template <class S, class ASrc, class WSrc>
__device__ __forceinline__ void mma4(const ASrc &as, const WSrc &ws, int k0, int k1, char *smem,
                                     f32x4 (&acc)[S::NB][S::MB])
{
    constexpr int MB = S::MB, NB = S::NB, AS = S::AS;
    constexpr int AB = S::A_BYTES, WB = S::W_BYTES;
    constexpr int AP = AB / 4096, WP = WB / 4096;  // copies per wave and step
    constexpr int NM = MB * NB, NF = MB + NB;
    constexpr uint32_t W0 = AS * AB;               // LDS: the A ring, then the W ring
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 1, wn = wave & 1, g = lane >> 4, x = lane & 15;

    typename ASrc::Row arow[AP];
    typename WSrc::Row wrow[WP];
#pragma unroll
    for (int i = 0; i < AP; ++i) {
        const int r = (wave * AP + i) * 8 + (lane >> 3);
        arow[i] = as.row(r, swz(r, lane & 7));
    }
#pragma unroll
    for (int i = 0; i < WP; ++i) {
        const int r = (wave * WP + i) * 8 + (lane >> 3);
        wrow[i] = ws.row(r, swz(r, lane & 7));
    }
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char *)smem;
    const uint32_t la0 = __builtin_amdgcn_readfirstlane(lds0 + wave * AP * 1024);
    const uint32_t lw0 = __builtin_amdgcn_readfirstlane(lds0 + wave * WP * 1024);
    auto copy_a = [&](const typename ASrc::Addr &ad, int i, uint32_t so) { as.copy(ad, la0 + so + i * 1024); };
    auto copy_w = [&](int i, uint32_t so, const typename WSrc::Step &st) {
        ws.copy(ws.addr(wrow[i], st), lw0 + so + i * 1024);
    };

#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) acc[nb][mb] = f32x4{0.f, 0.f, 0.f, 0.f};

    bf16x8 fa[2][MB], fw[2][NB];
    const int ra = wm * 16 * MB + x, rw = wn * 16 * NB + x;
    // fragment f (W's first) of half ks from A stage ao and W stage wo
    auto rd = [&](uint32_t ao, uint32_t wo, int ks, int f) {
        const lds_char *s = (const lds_char *)smem;
        if (f < NB)
            fw[ks][f] = *(const lds_bf16x8 *)(s + wo + (rw + f * 16) * kRowBytes + swz(rw, ks * 4 + g) * 16);
        else
            fa[ks][f - NB] = *(const lds_bf16x8 *)(s + ao + (ra + (f - NB) * 16) * kRowBytes + swz(ra, ks * 4 + g) * 16);
    };
    auto mfma2 = [&](int ks, int i) {
#pragma unroll
        for (int j = i; j < i + 2; ++j) mfma_into<S>(acc[j % NB][j / NB], fw[ks][j % NB], fa[ks][j / NB]);
    };

    const int kl = k1 - 1;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const auto sa = as.at(min(k0 + s, kl));
        const auto sw = ws.at(min(k0 + s, kl));
#pragma unroll
        for (int i = 0; i < AP; ++i) copy_a(as.addr(arow[i], sa), i, s * AB);
#pragma unroll
        for (int i = 0; i < WP; ++i) copy_w(i, W0 + s * WB, sw);
    }
    __asm__ volatile("s_waitcnt vmcnt(%0)" : : "n"(AP + WP) : "memory");
    __builtin_amdgcn_s_barrier();
    __asm__ volatile("" : : : "memory");
#pragma unroll
    for (int f = 0; f < NF; ++f) rd(0, W0, 0, f);

    constexpr int RD = NM * 3 / 4;  // a half's reads are spread over this many MFMAs
    uint32_t ao = 0, wo = W0;
    for (int kt = k0; kt < k1; ++kt) {
        const auto sa = as.at(min(kt + 2, kl));
        const auto sw = ws.at(min(kt + 2, kl));
        const uint32_t ao1 = ao + AB == AS * AB ? 0 : ao + AB, wo1 = wo == W0 ? W0 + WB : W0;
        const uint32_t ao2 = ao1 + AB == AS * AB ? 0 : ao1 + AB;
        typename ASrc::Addr ad{};
        // first half; with three A stages, A of step kt + 2 goes where step
        // kt - 1's was (its last read lies before the previous barrier)
#pragma unroll
        for (int i = 0; i < NM; i += 2) {
#pragma unroll
            for (int f = 0; f < NF; ++f)
                if (f * RD / NF / 2 * 2 == i) rd(ao, wo, 1, f);
            if constexpr (AS == 3) {
                // a copy's address is formed two MFMAs before the copy
#pragma unroll
                for (int l = 0; l < AP; ++l) {
                    const int at = (l * NM / AP + 2) / 2 * 2;
                    if (at == i) copy_a(ad, l, ao2);
                }
#pragma unroll
                for (int l = 0; l < AP; ++l) {
                    const int at = (l * NM / AP + 2) / 2 * 2;
                    if (at == i + 2) ad = as.addr(arow[l], sa);
                }
            }
            mfma2(0, i);
            __builtin_amdgcn_sched_barrier(0);
        }
        // step kt + 1 has landed, and every wave has read all of step kt
        __asm__ volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" : : "n"(AS == 3 ? AP : 0) : "memory");
        __builtin_amdgcn_s_barrier();
        __asm__ volatile("" : : : "memory");
        // second half; W of step kt + 2 (and A with two stages) replaces step kt's
        constexpr int NC = AS == 3 ? WP : AP + WP;
#pragma unroll
        for (int i = 0; i < NM; i += 2) {
#pragma unroll
            for (int f = 0; f < NF; ++f)
                if (f * RD / NF / 2 * 2 == i) rd(ao1, wo1, 0, f);
#pragma unroll
            for (int l = 0; l < NC; ++l)
                if (l * RD / NC / 2 * 2 == i) {
                    if (AS == 3 || l >= AP)
                        copy_w(AS == 3 ? l : l - AP, wo, sw);
                    else
                        copy_a(as.addr(arow[l], sa), l, ao);
                }
            mfma2(1, i);
            __builtin_amdgcn_sched_barrier(0);
        }
        ao = ao1, wo = wo1;
    }
    // wait states between the last MFMAs and the first read of their results
    if constexpr (S::WPE == 1) {
        __asm__ volatile("s_nop 15\n\ts_nop 15" : : : "memory");
        __builtin_amdgcn_sched_barrier(0);
    }
    wait_all_copies();
}

// An accumulator's value for the epilogue, by explicit moves where mfma_into
// is an instruction of its own: no other code then touches those registers,
// so that none can be placed (a copy, a spill) between the last MFMAs and the
// wait states that end mma4.  build.py reads the assembly of these kernels and
// refuses one that spills, or touches an accumulator near its MFMAs.
template <class S>
__device__ __forceinline__ f32x4 acc_value(f32x4 &a)
{
    if constexpr (S::WPE == 1) {
        f32x4 v;
        __asm__ volatile("v_accvgpr_read_b32 %0, %4\n\tv_accvgpr_read_b32 %1, %5\n\t"
                         "v_accvgpr_read_b32 %2, %6\n\tv_accvgpr_read_b32 %3, %7"
                         : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3])
                         : "a"(a[0]), "a"(a[1]), "a"(a[2]), "a"(a[3]));
        return v;
    } else {
        return a;
    }
}

// Activation of an epilogue.
template <int EPI>
__device__ __forceinline__ float activate(float y)
{
    return EPI == kBiasGelu ? gelu_tanh(y) : EPI == kBiasSilu ? silu(y) : y;
}

__device__ __forceinline__ f32x4 load_bias4(const uint16_t *bias, int n)
{
    f32x4 bv = {0.f, 0.f, 0.f, 0.f};
    if (bias != nullptr) {
        const uint64_t b4 = *reinterpret_cast<const uint64_t *>(bias + n);
#pragma unroll
        for (int i = 0; i < 4; ++i) bv[i] = bf((uint16_t)(b4 >> (16 * i)));
    }
    return bv;
}

// Writes a tile (m0, n0) from the accumulators of mma4.  A tile of whole
// width with 16-byte rows goes through the idle LDS, so that each store
// writes whole 16-byte chunks of consecutive rows (the fp32 residual in two
// halves of the channels); other tiles and split-K partials are written
// straight from the accumulators.  sp: K range of a kPartial launch.
template <class S, int EPI>
__device__ __forceinline__ void store4(const Out &o, int m0, int n0, int sp, char *smem, f32x4 (&acc)[S::NB][S::MB])
{
    constexpr int MB = S::MB, NB = S::NB, BM = S::BM, BN = S::BN;
    constexpr bool BF16_OUT = EPI == kBias || EPI == kBiasGelu || EPI == kBiasSilu;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 1, wn = wave & 1, g = lane >> 4, x = lane & 15;
    const bool whole = n0 + BN <= o.N && (reinterpret_cast<uintptr_t>(o.out) & 15) == 0 && (o.ldo & 7) == 0;
    if constexpr (BF16_OUT) {
        if (whole) {
            constexpr int CH = BN / 8;  // 16-byte chunks per staged row, chunk c of row r at c ^ (r & 7)
            static_assert(CH % 8 == 0 && (BM * CH) % kThreads4 == 0 && BM * BN * 2 <= S::LDS, "staging shape");
            __syncthreads();  // every wave is done with the rings
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const f32x4 bv = load_bias4(o.bias, n0 + wn * (16 * NB) + nb * 16 + 4 * g);
                const int c = wn * 2 * NB + nb * 2 + g / 2;
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) {
                    const int r = wm * 16 * MB + mb * 16 + x;
                    const f32x4 y = acc_value<S>(acc[nb][mb]) + bv;
                    bf16x4 w;
#pragma unroll
                    for (int i = 0; i < 4; ++i) w[i] = (__bf16)activate<EPI>(y[i]);
                    *(__attribute__((address_space(3))) bf16x4 *)((lds_char *)smem + r * (BN * 2) +
                                                                 ((c ^ (r & 7)) * 16) + (g & 1) * 8) = w;
                }
            }
            __syncthreads();
#pragma unroll 8
            for (int it = 0; it < BM * CH / kThreads4; ++it) {
                const int id = it * kThreads4 + (int)threadIdx.x;
                const int r = id / CH, c = id % CH;
                const bf16x8 v = *(const lds_bf16x8 *)((const lds_char *)smem + r * (BN * 2) + ((c ^ (r & 7)) * 16));
                if (m0 + r < o.M)
                    *reinterpret_cast<bf16x8 *>(static_cast<uint16_t *>(o.out) + (int64_t)(m0 + r) * o.ldo + n0 +
                                                c * 8) = v;
            }
            return;
        }
    }
    if constexpr (EPI == kGatedRes) {
        if (whole) {
            constexpr int HALF = BN / 2;  // channels per pass: one wave column
            constexpr int CH = HALF / 4;  // 16-byte chunks per staged row
            constexpr int NT = BM * CH / kThreads4, BT = NT % 8 == 0 ? 8 : NT % 6 == 0 ? 6 : NT % 5 == 0 ? 5 : 4;
            static_assert(CH % 8 == 0 && (BM * CH) % kThreads4 == 0 && BM * HALF * 4 <= S::LDS && NT % BT == 0,
                          "staging shape");
#pragma unroll
            for (int pass = 0; pass < 2; ++pass) {
                __syncthreads();  // the rings (first pass) or the previous half are no longer read
                if (wn == pass) {
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) {
                        const f32x4 bv = load_bias4(o.bias, n0 + wn * HALF + nb * 16 + 4 * g);
                        const int c = nb * 4 + g;
#pragma unroll
                        for (int mb = 0; mb < MB; ++mb) {
                            const int r = wm * 16 * MB + mb * 16 + x;
                            *(__attribute__((address_space(3))) f32x4 *)((lds_char *)smem + r * (HALF * 4) +
                                                                        ((c ^ (r & 7)) * 16)) = acc_value<S>(acc[nb][mb]) + bv;
                        }
                    }
                }
                __syncthreads();
                // BT chunks of the residual are requested before the first is used
                for (int t0 = 0; t0 < NT; t0 += BT) {
                    f32x4 res[BT];
#pragma unroll
                    for (int t = 0; t < BT; ++t) {
                        const int id = (t0 + t) * kThreads4 + (int)threadIdx.x;
                        const int r = id / CH, n = n0 + pass * HALF + (id % CH) * 4;
                        res[t] = *reinterpret_cast<const f32x4 *>(static_cast<const float *>(o.out) +
                                                                  (int64_t)min(m0 + r, o.M - 1) * o.ldo + n);
                    }
#pragma unroll
                    for (int t = 0; t < BT; ++t) {
                        const int id = (t0 + t) * kThreads4 + (int)threadIdx.x;
                        const int r = id / CH, c = id % CH, n = n0 + pass * HALF + c * 4;
                        const f32x4 y = *(const __attribute__((address_space(3))) f32x4 *)((const lds_char *)smem +
                                                                                         r * (HALF * 4) +
                                                                                         ((c ^ (r & 7)) * 16));
                        const f32x4 gv = o.gate != nullptr ? *reinterpret_cast<const f32x4 *>(o.gate + n)
                                                           : f32x4{1.f, 1.f, 1.f, 1.f};
                        if (m0 + r < o.M)
                            *reinterpret_cast<f32x4 *>(static_cast<float *>(o.out) + (int64_t)(m0 + r) * o.ldo + n) =
                                res[t] + gv * y;
                    }
                }
            }
            return;
        }
    }
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const int n = n0 + wn * (16 * NB) + nb * 16 + 4 * g;
        if (n >= o.N) continue;
        const f32x4 bv = EPI == kPartial ? f32x4{0.f, 0.f, 0.f, 0.f} : load_bias4(o.bias, n);
        f32x4 gv = {1.f, 1.f, 1.f, 1.f};
        if (EPI == kGatedRes && o.gate != nullptr) gv = *reinterpret_cast<const f32x4 *>(o.gate + n);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            const int m = m0 + wm * 16 * MB + mb * 16 + x;
            if (m >= o.M) continue;
            const f32x4 y = acc_value<S>(acc[nb][mb]) + bv;
            if constexpr (EPI == kPartial) {
                *reinterpret_cast<f32x4 *>(static_cast<float *>(o.out) + ((int64_t)sp * o.M + m) * o.ldo + n) = y;
            } else if constexpr (EPI == kGatedRes) {
                f32x4 *p = reinterpret_cast<f32x4 *>(static_cast<float *>(o.out) + (int64_t)m * o.ldo + n);
                *p = *p + gv * y;
            } else {
                bf16x4 w;
#pragma unroll
                for (int i = 0; i < 4; ++i) w[i] = (__bf16)activate<EPI>(y[i]);
                *reinterpret_cast<bf16x4 *>(static_cast<uint16_t *>(o.out) + (int64_t)m * o.ldo + n) = w;
            }
        }
    }
}

inline int tiles_along(int n, int b)
{
    return (n + b - 1) / b;
}

}  // namespace tile
}  // namespace regenvc
