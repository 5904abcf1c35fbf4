// LayerNorm-side transposition for the Shfl-BW kernels on gfx950 (CDNA4).
//
// The sparse kernels read and write their dense matrices row-wise, so they
// want activations batch-innermost: X[K features][N tokens].  A LayerNorm
// produces them feature-innermost, x[N][K]; Section 4.3 (discussion of the
// activation layout) folds the transposition into that LayerNorm.  This
// kernel is that step: per token it normalises over the K features (mean,
// biased variance, eps, then gamma and beta), or just copies when asked to,
// and writes the result transposed.
//
// A workgroup (8 wavefronts) owns 64 tokens and a range of the features.
// Phase A: each wavefront takes 8 tokens and sums x - p and (x - p)^2 over
// all K features in one sweep, p being the token's first feature (a pivot
// near the data keeps the fp32 variance free of cancellation); 16 row loads
// are in flight per lane.  Workgroups that share tokens repeat this sweep;
// all but the first read it from the L2.  Phase B: 64-feature blocks of the
// workgroup's range are loaded up to four blocks ahead (16 bytes per lane),
// normalised in fp32, written transposed into an LDS tile and stored as 64
// rows of 128 bytes.  It is bound by HBM: 2*N*K bytes read and 2*N*K written.
//
// When a block of 32 (or 64) tokens with all its features fits the LDS, a
// second kernel keeps it there instead: every activation is read from HBM
// once, the statistics come from the same loads (sixteen wavefronts, two or four
// tokens each),
// and the transposed rows are gathered from LDS columns, two neighbouring
// features per lane (row pitch chosen so that the 64 four-byte reads of a
// wavefront fall into 64 different banks).  Rows too wide for that go through registers, 1024 features
// at a time; few tokens have their features shared by several workgroups (layernorm_transpose_few_kernel).
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "choice.h"
#include "shflbw.h"
#include "shflbw_internal.h"

namespace shflbw {
namespace {

typedef unsigned short ln_ushort8 __attribute__((ext_vector_type(8)));

constexpr int LN_TOK = 64;       // tokens per workgroup
constexpr int LN_WAVES = 8;
constexpr int LN_FB = 64;        // features per block in phase B
constexpr int LN_PITCH = LN_TOK + 8;   // LDS row pitch of the transposed tile (16-bit units)
constexpr int LN_AHEAD = 4;      // feature blocks loaded ahead

struct LnArgs {
    const uint16_t* x;      // [N][K], leading dimension ldx
    const uint16_t* gamma;  // [K] or nullptr
    const uint16_t* beta;   // [K] or nullptr
    uint16_t* out;          // [K][N], leading dimension ldo
    long ldx, ldo, N;
    int K;
    float eps;
    int normalize;
    int stream;             // streaming stores, see ln_store
    int blocks_per_wg;      // 64-feature blocks one workgroup transposes (grid.y covers K)
    int slices_per_wg;      // register-resident variant: 1024-feature slices one workgroup stores (grid.y covers K)
};

// the kernel for few tokens
struct LnFew {
    int blocks, slice, pitch;   // token blocks; features of a slice; LDS pitch of a token's slice, 16-bit units
    int per_xcd, total;         // workgroups of an XCD, and with work
};

// Streaming where the row segments of 64 (128) bytes are whole 64-byte blocks of memory; plain where
// two workgroups share a block, so that its parts meet in the L2 (8184 tokens of 1024 features: 16.0 us
// streaming, 11.0 plain; 20 008 of 1024: 41 and 26; 8192 of 1024: 8.2 and 8.9).
template <bool STREAM>
__device__ __forceinline__ void ln_store(uint16_t* p, ln_ushort8 v)
{
    if constexpr (STREAM) __builtin_nontemporal_store(v, reinterpret_cast<ln_ushort8*>(p));
    else *reinterpret_cast<ln_ushort8*>(p) = v;
}
// f with std::true_type or std::false_type, once for many stores: a choice at each of them keeps the loop around
// them from being unrolled (32 768 tokens of 256 features, transposed only: 5.9 us against 5.2)
template <class F>
__device__ __forceinline__ void ln_with_stores(int stream, F&& f)
{
    if (stream) {
        asm volatile("");   // kept apart: merged with the other branch, the stores lose their hint
        f(std::true_type{});
        asm volatile("");
    } else {
        f(std::false_type{});
    }
}

template <bool BF>
__device__ __forceinline__ float ln_widen(uint16_t v)
{
    if constexpr (BF) return __builtin_bit_cast(float, (unsigned)v << 16);
    else return (float)__builtin_bit_cast(_Float16, v);
}
template <bool BF>
__device__ __forceinline__ uint16_t ln_narrow(float f)
{
    if constexpr (BF) return __builtin_bit_cast(uint16_t, (__bf16)f);
    else return __builtin_bit_cast(uint16_t, (_Float16)f);
}

template <bool BF, bool NORM>
__global__ __launch_bounds__(64 * LN_WAVES) void layernorm_transpose_kernel(LnArgs a)
{
    __shared__ float stat_mean[LN_TOK], stat_rstd[LN_TOK];
    __shared__ __attribute__((aligned(16))) uint16_t tile[LN_FB * LN_PITCH];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const long n0 = (long)blockIdx.x * LN_TOK;
    const int K = a.K;

    // phase B's first blocks are requested now, so that they travel while phase A runs
    // load: thread -> token tid/8, 8 features at (tid%8)*8 of the block;
    // store: thread -> feature row tid/8 of the block, 8 tokens at (tid%8)*8
    const int ltok = tid >> 3, lchunk = tid & 7;
    const int nblocks_all = (K + LN_FB - 1) / LN_FB;
    const int bbeg = blockIdx.y * a.blocks_per_wg;
    int bend = bbeg + a.blocks_per_wg;
    bend = bend < nblocks_all ? bend : nblocks_all;
    const long ntok = n0 + ltok;
    auto load_block = [&](int b, ln_ushort8& v) __attribute__((always_inline)) {
        const int k = b * LN_FB + lchunk * 8;
        v = ln_ushort8{0, 0, 0, 0, 0, 0, 0, 0};
        if (b < bend && k < K && ntok < a.N) v = *reinterpret_cast<const ln_ushort8*>(a.x + ntok * a.ldx + k);
    };
    ln_ushort8 ring[LN_AHEAD];
#pragma unroll
    for (int u = 0; u < LN_AHEAD; ++u) load_block(bbeg + u, ring[u]);

    // ---------------------------------------------------------------- phase A
    if (NORM) {
        constexpr int TPW = LN_TOK / LN_WAVES;   // tokens per wavefront
        float s1[TPW], s2[TPW], pivot[TPW];
#pragma unroll
        for (int t = 0; t < TPW; ++t) { s1[t] = 0.f; s2[t] = 0.f; pivot[t] = 0.f; }
        for (int kc0 = 0; kc0 < K; kc0 += 2 * 64 * 8) {
            ln_ushort8 v[TPW][2];
#pragma unroll
            for (int t = 0; t < TPW; ++t) {
                const long n = n0 + wave * TPW + t;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int kc = kc0 + h * 512 + lane * 8;
                    v[t][h] = ln_ushort8{0, 0, 0, 0, 0, 0, 0, 0};
                    if (n < a.N && kc < K) v[t][h] = *reinterpret_cast<const ln_ushort8*>(a.x + n * a.ldx + kc);
                }
            }
            if (kc0 == 0) {
                // the token's first feature, which lane 0 has just loaded
#pragma unroll
                for (int t = 0; t < TPW; ++t)
                    pivot[t] = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(
                        __builtin_bit_cast(int, ln_widen<BF>(v[t][0][0]))));
            }
#pragma unroll
            for (int t = 0; t < TPW; ++t) {
                const long n = n0 + wave * TPW + t;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int kc = kc0 + h * 512 + lane * 8;
                    if (n < a.N && kc < K) {
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            const float d = ln_widen<BF>(v[t][h][e]) - pivot[t];
                            s1[t] += d;
                            s2[t] += d * d;
                        }
                    }
                }
            }
        }
#pragma unroll
        for (int t = 0; t < TPW; ++t) {
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) {
                s1[t] += __shfl_xor(s1[t], off, 64);
                s2[t] += __shfl_xor(s2[t], off, 64);
            }
        }
        if (lane == 0) {
#pragma unroll
            for (int t = 0; t < TPW; ++t) {
                const float m = s1[t] / (float)K;              // mean of x - pivot
                float var = s2[t] / (float)K - m * m;
                var = var > 0.f ? var : 0.f;
                stat_mean[wave * TPW + t] = pivot[t] + m;
                stat_rstd[wave * TPW + t] = 1.0f / __builtin_sqrtf(var + a.eps);
            }
        }
    } else if (tid < LN_TOK) {
        stat_mean[tid] = 0.f;
        stat_rstd[tid] = 1.f;
    }
    __syncthreads();

    // ---------------------------------------------------------------- phase B
    const float mean = stat_mean[ltok], rstd = stat_rstd[ltok];

    for (int b0 = bbeg; b0 < bend; b0 += LN_AHEAD) {
#pragma unroll
        for (int u = 0; u < LN_AHEAD; ++u) {
            const int b = b0 + u;
            if (b < bend) {   // uniform
                const int k = b * LN_FB + lchunk * 8;
                if (NORM) {
                    float g[8], bt[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) { g[e] = 1.f; bt[e] = 0.f; }
                    if (k < K) {
                        if (a.gamma) {
                            const ln_ushort8 gv = *reinterpret_cast<const ln_ushort8*>(a.gamma + k);
#pragma unroll
                            for (int e = 0; e < 8; ++e) g[e] = ln_widen<BF>(gv[e]);
                        }
                        if (a.beta) {
                            const ln_ushort8 bv = *reinterpret_cast<const ln_ushort8*>(a.beta + k);
#pragma unroll
                            for (int e = 0; e < 8; ++e) bt[e] = ln_widen<BF>(bv[e]);
                        }
                    }
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        tile[(lchunk * 8 + e) * LN_PITCH + ltok] =
                            ln_narrow<BF>((ln_widen<BF>(ring[u][e]) - mean) * rstd * g[e] + bt[e]);
                } else {
#pragma unroll
                    for (int e = 0; e < 8; ++e) tile[(lchunk * 8 + e) * LN_PITCH + ltok] = ring[u][e];
                }
                load_block(b + LN_AHEAD, ring[u]);
                __syncthreads();
                {
                    const int kr = ltok;   // the same split of the thread index, now feature row / token chunk
                    const long kk = (long)b * LN_FB + kr, n = n0 + lchunk * 8;
                    if (kk < K && n < a.N)
                        *reinterpret_cast<ln_ushort8*>(a.out + kk * a.ldo + n) =
                            *reinterpret_cast<const ln_ushort8*>(tile + kr * LN_PITCH + lchunk * 8);
                }
                __syncthreads();
            }
        }
    }
}

// ---------------------------------------------------------------- LDS-resident variant
// TOK tokens x K features (pitch P halves) + statistics + gamma/beta in fp32.  A lane of
// the store phase takes two neighbouring features of 8 tokens: 8 four-byte LDS reads
// for two 16-byte stores.  The 64 lanes of a wavefront read, per token, 64/CH feature
// pairs for each of CH token chunks; with P/2 = 64/CH/8 (mod 8) the chunks' rows start
// 64/CH banks apart, so the 64 words fall into 64 different banks.
// lo = low half of w + c, hi = high half of w + c, in fp32.  For float16 the widening
// rides on the mixed-precision multiply-add (x * 1 + c, rounded once: the same bits as
// a conversion followed by an addition), which halves the instructions.
template <bool BF>
__device__ __forceinline__ void ln_add_pair(unsigned w, float c, float& lo, float& hi)
{
    if constexpr (BF) {
        lo = __builtin_bit_cast(float, w << 16) + c;
        hi = __builtin_bit_cast(float, w & 0xffff0000u) + c;
    } else {
        asm("v_fma_mix_f32 %0, %1, 1.0, %2 op_sel_hi:[1,0,0]" : "=v"(lo) : "v"(w), "v"(c));
        asm("v_fma_mix_f32 %0, %1, 1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(hi) : "v"(w), "v"(c));
    }
}

template <bool BF, int TOK, bool NORM>
__global__ __launch_bounds__(1024) void layernorm_transpose_resident_kernel(LnArgs a, int P)
{
    extern __shared__ __attribute__((aligned(16))) char ln_smem[];
    uint16_t* xs = reinterpret_cast<uint16_t*>(ln_smem);                       // [TOK][P]
    float* st_mean = reinterpret_cast<float*>(ln_smem + (size_t)TOK * P * 2);   // [TOK]
    float* st_rstd = st_mean + TOK;                                             // [TOK]
    float* gam = st_rstd + TOK;                                                 // [K]
    float* bet = gam + a.K;                                                     // [K]
    constexpr int WAVES = 16;
    constexpr int TPW = TOK / WAVES;     // tokens per wavefront: 2 or 4
    constexpr int CH = TOK / 8;           // 16-byte token chunks per output row
    constexpr int FP = 64 / CH;           // feature pairs one wavefront stores per pass
    constexpr bool WIDE = (TOK == 32);    // its pitch keeps every row 8-byte aligned

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const long n0 = (long)blockIdx.x * TOK;
    const int K = a.K;

    if (NORM) {
        for (int k = tid; k < K; k += 64 * WAVES) {
            gam[k] = a.gamma ? ln_widen<BF>(a.gamma[k]) : 1.f;
            bet[k] = a.beta ? ln_widen<BF>(a.beta[k]) : 0.f;
        }
    }

    // ---- load the block once: LDS copy and, from the same registers, the statistics
    float s1[TPW], s2[TPW], pivot[TPW];
#pragma unroll
    for (int t = 0; t < TPW; ++t) { s1[t] = 0.f; s2[t] = 0.f; pivot[t] = 0.f; }
    const bool all_tokens = n0 + TOK <= a.N;
    // one sweep of HALVES times 512 features; FULL = every token and feature of it exists
    auto sweep = [&](int kc0, auto full_tag, auto halves_tag) __attribute__((always_inline)) {
        constexpr bool FULL = decltype(full_tag)::value;
        constexpr int HALVES = decltype(halves_tag)::value;
        ln_ushort8 v[TPW][HALVES];
#pragma unroll
        for (int t = 0; t < TPW; ++t) {
            const long n = n0 + wave * TPW + t;
#pragma unroll
            for (int h = 0; h < HALVES; ++h) {
                const int kc = kc0 + h * 512 + lane * 8;
                // a token or feature that does not exist loads the last one instead (its values are neither
                // summed, nor kept, nor stored: a conditional load would wait for the one before it)
                const long nc = FULL || n < a.N ? n : a.N - 1;
                const int cc = FULL || kc < K ? kc : K - 8;
                v[t][h] = *reinterpret_cast<const ln_ushort8*>(a.x + nc * a.ldx + cc);
            }
        }
        if (NORM && kc0 == 0) {
#pragma unroll
            for (int t = 0; t < TPW; ++t)
                pivot[t] = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(
                    __builtin_bit_cast(int, ln_widen<BF>(v[t][0][0]))));
        }
#pragma unroll
        for (int t = 0; t < TPW; ++t) {
#pragma unroll
            for (int h = 0; h < HALVES; ++h) {
                const int kc = kc0 + h * 512 + lane * 8;
                if (FULL || kc < K) {
                    unsigned w[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        w[e] = (unsigned)v[t][h][2 * e] | ((unsigned)v[t][h][2 * e + 1] << 16);
                    uint16_t* row = xs + (wave * TPW + t) * P + kc;
                    if (WIDE) {
                        uint2* dst = reinterpret_cast<uint2*>(row);
                        dst[0] = uint2{w[0], w[1]};
                        dst[1] = uint2{w[2], w[3]};
                    } else {
                        unsigned* dst = reinterpret_cast<unsigned*>(row);
#pragma unroll
                        for (int e = 0; e < 4; ++e) dst[e] = w[e];
                    }
                    if (NORM) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            float d0, d1;
                            ln_add_pair<BF>(w[e], -pivot[t], d0, d1);
                            s1[t] += d0;
                            s2[t] += d0 * d0;
                            s1[t] += d1;
                            s2[t] += d1 * d1;
                        }
                    }
                }
            }
        }
    };
    // 512 features or fewer: the second half would load the last ones over and over (32 768 tokens of 256, transposed
    // only, 5.9 us without this, 4.5 with it)
    if (K <= 64 * 8) sweep(0, std::false_type{}, std::integral_constant<int, 1>{});
    else
        for (int kc0 = 0; kc0 < K; kc0 += 2 * 64 * 8) {
            if (all_tokens && kc0 + 2 * 64 * 8 <= K) sweep(kc0, std::true_type{}, std::integral_constant<int, 2>{});
            else sweep(kc0, std::false_type{}, std::integral_constant<int, 2>{});
        }
    if (NORM) {
#pragma unroll
        for (int t = 0; t < TPW; ++t) {
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) {
                s1[t] += __shfl_xor(s1[t], off, 64);
                s2[t] += __shfl_xor(s2[t], off, 64);
            }
        }
        if (lane == 0) {
#pragma unroll
            for (int t = 0; t < TPW; ++t) {
                const float m = s1[t] / (float)K;
                float var = s2[t] / (float)K - m * m;
                var = var > 0.f ? var : 0.f;
                st_mean[wave * TPW + t] = pivot[t] + m;
                st_rstd[wave * TPW + t] = 1.0f / __builtin_sqrtf(var + a.eps);
            }
        }
    }
    __syncthreads();

    // ---- transposed rows: a wavefront stores 2*FP feature rows x TOK tokens per pass;
    // lane -> features 2*(lane/CH), +1 of the pass, tokens (lane%CH)*8 .. +7
    const int kk2 = lane / CH, tchunk = lane % CH;
    float mean[8], rstd[8];
    if (NORM) {
#pragma unroll
        for (int e = 0; e < 8; ++e) { mean[e] = st_mean[tchunk * 8 + e]; rstd[e] = st_rstd[tchunk * 8 + e]; }
    }
    const long n = n0 + tchunk * 8;
    const unsigned* xw = reinterpret_cast<const unsigned*>(xs) + tchunk * 8 * (P / 2);
    const int Q = P / 2;
    if (n < a.N) {
        ln_with_stores(a.stream, [&](auto stream_tag) __attribute__((always_inline)) {
            constexpr bool STREAM = decltype(stream_tag)::value;
#pragma unroll 2
            for (int kb = wave * 2 * FP; kb < K; kb += WAVES * 2 * FP) {
                const int k = kb + 2 * kk2;      // K is even: the pair exists or does not
                if (k < K) {
                    unsigned w[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) w[e] = xw[e * Q + (k >> 1)];
                    ln_ushort8 o0, o1;
                    if (NORM) {
                        const float2 g = *reinterpret_cast<const float2*>(gam + k);
                        const float2 b = *reinterpret_cast<const float2*>(bet + k);
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            float lo, hi;
                            ln_add_pair<BF>(w[e], -mean[e], lo, hi);
                            o0[e] = ln_narrow<BF>(lo * rstd[e] * g.x + b.x);
                            o1[e] = ln_narrow<BF>(hi * rstd[e] * g.y + b.y);
                        }
                    } else {
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            o0[e] = (uint16_t)(w[e] & 0xffffu);
                            o1[e] = (uint16_t)(w[e] >> 16);
                        }
                    }
                    uint16_t* dst = a.out + (long)k * a.ldo + n;
                    ln_store<STREAM>(dst, o0);
                    ln_store<STREAM>(dst + a.ldo, o1);
                }
            }
        });
    }
}

// ---------------------------------------------------------------- register-resident variant
// For feature counts whose token blocks no longer fit the LDS: a workgroup of sixteen
// wavefronts keeps 4096 features of its 32 tokens in registers (two tokens per wavefront,
// 64 registers per lane), takes the statistics from there, and passes them through the
// LDS in slices of 1024 features, double-buffered so that one barrier per slice suffices;
// the transposed store of a slice is the LDS-resident kernel's.  Up to 4096 features
// (PARTS = 1) every activation is read from HBM once.  Wider rows (PARTS = 2 .. 4, up to
// 16384 features) are swept in parts of 4096 for the statistics; the last part stays in
// registers and goes out first, the others are read again (2 - 1/PARTS reads per
// activation; the streaming kernel reads a row once per workgroup that shares its
// tokens, and 16-token blocks, whose 32-byte row segments halve the write rate, measured
// 187 us against 112 on 8192 x 8192).
// SHARED: several workgroups (grid.y) share a token block; each takes the statistics for itself and
// stores its own slices, which it reads again.
template <bool BF, bool NORM, int PARTS, bool SHARED>
__global__ __launch_bounds__(1024) void layernorm_transpose_register_kernel(LnArgs a)
{
    constexpr int TOK = 32, WAVES = 16, TPW = 2, KH = 4096, SL = 1024, NSL = KH / SL;
    constexpr int CH = TOK / 8, FP = 64 / CH;
    constexpr int P = SL + 4, Q = P / 2;   // Q = 2 (mod 8): see the LDS-resident kernel
    extern __shared__ __attribute__((aligned(16))) char ln_smem[];
    uint16_t* xs = reinterpret_cast<uint16_t*>(ln_smem);                          // [2][TOK][P]
    float* st_mean = reinterpret_cast<float*>(ln_smem + (size_t)2 * TOK * P * 2);  // [TOK]
    float* st_rstd = st_mean + TOK;                                                // [TOK]

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const long n0 = (long)blockIdx.x * TOK;
    const int K = a.K;
    const bool full = n0 + TOK <= a.N && K == KH * PARTS;

    // chunk j of a token's part: features part*4096 + j*512 + lane*8 .. +7
    ln_ushort8 v[TPW][2 * NSL];
    float s1[TPW], s2[TPW], pivot[TPW];
#pragma unroll
    for (int t = 0; t < TPW; ++t) { s1[t] = 0.f; s2[t] = 0.f; pivot[t] = 0.f; }
    auto fetch_as = [&](int part, auto full_tag, auto stats_tag) __attribute__((always_inline)) {
        constexpr bool FULL = decltype(full_tag)::value, STATS = decltype(stats_tag)::value;
        const int kh = part * KH;
#pragma unroll
        for (int t = 0; t < TPW; ++t) {
            const long n = n0 + wave * TPW + t;
#pragma unroll
            for (int j = 0; j < 2 * NSL; ++j) {
                const int kc = kh + j * 512 + lane * 8;
                // what does not exist loads the last token or feature (neither summed nor stored)
                const long nc = FULL || n < a.N ? n : a.N - 1;
                const int cc = FULL || kc < K ? kc : K - 8;
                v[t][j] = *reinterpret_cast<const ln_ushort8*>(a.x + nc * a.ldx + cc);
            }
        }
        if (STATS) {
#pragma unroll
            for (int t = 0; t < TPW; ++t) {
                if (part == 0)
                    pivot[t] = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(
                        __builtin_bit_cast(int, ln_widen<BF>(v[t][0][0]))));
#pragma unroll
                for (int j = 0; j < 2 * NSL; ++j) {
                    if (FULL || kh + j * 512 + lane * 8 < K) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const unsigned w = (unsigned)v[t][j][2 * e] | ((unsigned)v[t][j][2 * e + 1] << 16);
                            float d0, d1;
                            ln_add_pair<BF>(w, -pivot[t], d0, d1);
                            s1[t] += d0;
                            s2[t] += d0 * d0;
                            s1[t] += d1;
                            s2[t] += d1 * d1;
                        }
                    }
                }
            }
        }
    };
    auto fetch = [&](int part, auto stats_tag) __attribute__((always_inline)) {
        if (full) fetch_as(part, std::true_type{}, stats_tag);
        else fetch_as(part, std::false_type{}, stats_tag);
    };

    const int kk2 = lane / CH, tchunk = lane % CH;
    const long n = n0 + tchunk * 8;
    float mean[8], rstd[8];
    // 1.0 twice in the 16-bit format, for an absent gamma
    const unsigned one2 = BF ? 0x3f803f80u : 0x3c003c00u;
    // the transposed rows k0 .. k0+1023 from LDS buffer `buf`
    auto store_slice_as = [&](int k0, int buf, auto stream_tag) __attribute__((always_inline)) {
        const unsigned* xw = reinterpret_cast<const unsigned*>(xs + buf * TOK * P) + tchunk * 8 * Q;
#pragma unroll
        for (int pass = 0; pass < SL / (WAVES * 2 * FP); ++pass) {
            const int kl = (pass * WAVES + wave) * 2 * FP + 2 * kk2;   // feature inside the slice
            const int k = k0 + kl;
            if (k < K && n < a.N) {
                unsigned w[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) w[e] = xw[e * Q + (kl >> 1)];
                ln_ushort8 o0, o1;
                if (NORM) {
                    const unsigned gw = a.gamma ? *reinterpret_cast<const unsigned*>(a.gamma + k) : one2;
                    const unsigned bw = a.beta ? *reinterpret_cast<const unsigned*>(a.beta + k) : 0u;
                    float g0, g1, b0, b1;
                    ln_add_pair<BF>(gw, 0.f, g0, g1);
                    ln_add_pair<BF>(bw, 0.f, b0, b1);
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        float lo, hi;
                        ln_add_pair<BF>(w[e], -mean[e], lo, hi);
                        o0[e] = ln_narrow<BF>(lo * rstd[e] * g0 + b0);
                        o1[e] = ln_narrow<BF>(hi * rstd[e] * g1 + b1);
                    }
                } else {
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        o0[e] = (uint16_t)(w[e] & 0xffffu);
                        o1[e] = (uint16_t)(w[e] >> 16);
                    }
                }
                uint16_t* dst = a.out + (long)k * a.ldo + n;
                ln_store<decltype(stream_tag)::value>(dst, o0);
                ln_store<decltype(stream_tag)::value>(dst + a.ldo, o1);
            }
        }
    };
    auto store_slice = [&](int k0, int buf) __attribute__((always_inline)) {
        ln_with_stores(a.stream, [&](auto stream_tag) __attribute__((always_inline)) { store_slice_as(k0, buf, stream_tag); });
    };
    // the part held in registers, slice by slice through the LDS, out as transposed rows
    auto emit = [&](int part) __attribute__((always_inline)) {
        const int kh = part * KH;
        auto stage = [&](int sl) __attribute__((always_inline)) {
#pragma unroll
            for (int t = 0; t < TPW; ++t) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const ln_ushort8& c = v[t][2 * sl + h];
                    uint2* dst = reinterpret_cast<uint2*>(xs + ((sl & 1) * TOK + wave * TPW + t) * P + h * 512 + lane * 8);
                    dst[0] = uint2{(unsigned)c[0] | ((unsigned)c[1] << 16), (unsigned)c[2] | ((unsigned)c[3] << 16)};
                    dst[1] = uint2{(unsigned)c[4] | ((unsigned)c[5] << 16), (unsigned)c[6] | ((unsigned)c[7] << 16)};
                }
            }
        };
        // buffer 0's last readers passed the barrier that closed the slice before
        stage(0);
        __syncthreads();
#pragma unroll
        for (int sl = 0; sl < NSL; ++sl) {
            // whole slices every time (a slice beyond K stores nothing), so that every wavefront
            // meets every barrier
            if (sl + 1 < NSL) stage(sl + 1);
            store_slice(kh + sl * SL, sl & 1);
            __syncthreads();
        }
    };

    // SHARED: slices [sl, end) from memory, the next one in flight while one is stored
    auto emit_own = [&]() __attribute__((always_inline)) {
        int sl = blockIdx.y * a.slices_per_wg;
        const int all = (K + SL - 1) / SL, end = sl + a.slices_per_wg < all ? sl + a.slices_per_wg : all;
        ln_ushort8 c[TPW][2];
        auto request = [&](int s) __attribute__((always_inline)) {
#pragma unroll
            for (int t = 0; t < TPW; ++t) {
                const long nt = n0 + wave * TPW + t;
                const long nc = nt < a.N ? nt : a.N - 1;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int kc = s * SL + h * 512 + lane * 8;
                    c[t][h] = *reinterpret_cast<const ln_ushort8*>(a.x + nc * a.ldx + (kc < K ? kc : K - 8));
                }
            }
        };
        request(sl);
        for (; sl < end; ++sl) {
#pragma unroll
            for (int t = 0; t < TPW; ++t)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    uint2* dst = reinterpret_cast<uint2*>(xs + ((sl & 1) * TOK + wave * TPW + t) * P + h * 512 + lane * 8);
                    const ln_ushort8& w = c[t][h];
                    dst[0] = uint2{(unsigned)w[0] | ((unsigned)w[1] << 16), (unsigned)w[2] | ((unsigned)w[3] << 16)};
                    dst[1] = uint2{(unsigned)w[4] | ((unsigned)w[5] << 16), (unsigned)w[6] | ((unsigned)w[7] << 16)};
                }
            if (sl + 1 < end) request(sl + 1);
            __syncthreads();   // the slice is there; the buffer of the slice before last is free again
            store_slice(sl * SL, sl & 1);
        }
    };

    if (!NORM && SHARED) {
        emit_own();
        return;
    }
    if (!NORM) {
        // nothing to wait for: each part goes out as it comes in
#pragma unroll
        for (int part = 0; part < PARTS; ++part) {
            fetch(part, std::false_type{});
            emit(part);
        }
        return;
    }
#pragma unroll
    for (int part = 0; part < PARTS; ++part) fetch(part, std::true_type{});
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            s1[t] += __shfl_xor(s1[t], off, 64);
            s2[t] += __shfl_xor(s2[t], off, 64);
        }
    }
    if (lane == 0) {
#pragma unroll
        for (int t = 0; t < TPW; ++t) {
            const float m = s1[t] / (float)K;
            float var = s2[t] / (float)K - m * m;
            var = var > 0.f ? var : 0.f;
            st_mean[wave * TPW + t] = pivot[t] + m;
            st_rstd[wave * TPW + t] = 1.0f / __builtin_sqrtf(var + a.eps);
        }
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 8; ++e) { mean[e] = st_mean[tchunk * 8 + e]; rstd[e] = st_rstd[tchunk * 8 + e]; }
    if (SHARED) {
        emit_own();
        return;
    }
    emit(PARTS - 1);   // the part the sweep left in the registers
#pragma unroll
    for (int part = 0; part < PARTS - 1; ++part) {
        fetch(part, std::false_type{});
        emit(part);
    }
}

// Few tokens.  What bounds it is one chain of latencies, launch -> rows -> statistics -> rows of the output, and how long a CU
// takes over its part of each: with 32 tokens and all their features to a workgroup, most CUs had none and the others 2.4 us
// per 1024 features.  Here a workgroup reads the rows of TOK tokens (16 or 8: 64 KB at 2048 or 4096 features) once, into the
// registers of its sixteen wavefronts, takes the statistics, and passes on only a slice of the features (few.slice of them, a multiple
// of 16): every slice of a token block is another workgroup's, which reads the rows for itself, mostly from the L2.  Output rows get 32 or 16
// bytes per workgroup, half the write rate or less, which is why many tokens do not come here (the rule is where it is launched).
template <bool BF, int TOK>
__global__ __launch_bounds__(1024) void layernorm_transpose_few_kernel(LnArgs a, LnFew few)
{
    static_assert(TOK == 16 || TOK == 8, "whole tokens per wavefront, or two wavefronts per token");
    constexpr int WPT = 16 / TOK;                            // wavefronts of a token, which take its runs of 512 features in turn
    constexpr int RUNS = TOK == 16 ? 4 : 16;                 // of a wavefront, at most: 2048 features of 16 tokens, 16 384 of 8
    constexpr int CH = TOK / 8, FP = 64 / CH;
    extern __shared__ __attribute__((aligned(16))) char ln_smem[];
    const int P = few.pitch, Q = P / 2;
    uint16_t* xs = reinterpret_cast<uint16_t*>(ln_smem);     // [TOK][P]
    float* st_mean = reinterpret_cast<float*>(ln_smem + (size_t)TOK * P * 2);   // [TOK]
    float* st_rstd = st_mean + TOK;                          // [TOK]
    float* st_part = st_rstd + TOK;                          // [2][16]: sums of a wavefront, where a token has two

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // an XCD takes neighbouring token blocks of a slice: the parts of a 64-byte block that they write meet in its L2
    const unsigned w = (blockIdx.x & 7) * (unsigned)few.per_xcd + (blockIdx.x >> 3);
    if (w >= (unsigned)few.total) return;                    // uniform for the workgroup
    const int sl = (int)(w / (unsigned)few.blocks);
    const long n0 = (long)((int)w - sl * few.blocks) * TOK;
    const int K = a.K, k0 = sl * few.slice, k1 = k0 + few.slice < K ? k0 + few.slice : K;
    const int token = wave / WPT, run0 = wave % WPT;

    // what does not exist loads the last token or feature (neither summed nor stored)
    const long nt = n0 + token;
    const uint16_t* row = a.x + (nt < a.N ? nt : a.N - 1) * a.ldx;
    const uint16_t first = row[0];
    ln_ushort8 v[RUNS];
#pragma unroll
    for (int j = 0; j < RUNS; ++j) {
        const int kc = (j * WPT + run0) * 512 + lane * 8;
        if ((j * WPT + run0) * 512 < K)                      // uniform for the wavefront
            v[j] = *reinterpret_cast<const ln_ushort8*>(row + (kc < K ? kc : K - 8));
    }
    // the outputs' place, and gamma and beta of this lane's first features
    const int kk2 = lane / CH, tchunk = lane % CH;
    const long n = n0 + tchunk * 8;
    const unsigned one2 = BF ? 0x3f803f80u : 0x3c003c00u;    // 1.0 twice, for an absent gamma
    auto feature = [&](int pass) __attribute__((always_inline)) { return (pass * 16 + wave) * 2 * FP + 2 * kk2; };
    auto gamma_of = [&](int k) __attribute__((always_inline)) { return a.gamma ? *reinterpret_cast<const unsigned*>(a.gamma + (k < K ? k : K - 8)) : one2; };
    auto beta_of = [&](int k) __attribute__((always_inline)) { return a.beta ? *reinterpret_cast<const unsigned*>(a.beta + (k < K ? k : K - 8)) : 0u; };
    unsigned gw = gamma_of(k0 + feature(0)), bw = beta_of(k0 + feature(0));

    float s1 = 0.f, s2 = 0.f;
    const float pivot = ln_widen<BF>(first);
#pragma unroll
    for (int j = 0; j < RUNS; ++j) {
        const int kc = (j * WPT + run0) * 512 + lane * 8;
        if (kc < K) {
            const ln_ushort8& c = v[j];
            const unsigned p[4] = {(unsigned)c[0] | ((unsigned)c[1] << 16), (unsigned)c[2] | ((unsigned)c[3] << 16),
                                   (unsigned)c[4] | ((unsigned)c[5] << 16), (unsigned)c[6] | ((unsigned)c[7] << 16)};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float d0, d1;
                ln_add_pair<BF>(p[e], -pivot, d0, d1);
                s1 += d0;
                s2 += d0 * d0;
                s1 += d1;
                s2 += d1 * d1;
            }
            if (kc >= k0 && kc < k1) {
                uint2* dst = reinterpret_cast<uint2*>(xs + token * P + kc - k0);
                dst[0] = uint2{p[0], p[1]};
                dst[1] = uint2{p[2], p[3]};
            }
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        s1 += __shfl_xor(s1, off, 64);
        s2 += __shfl_xor(s2, off, 64);
    }
    if constexpr (WPT == 2) {
        if (lane == 0) { st_part[wave] = s1; st_part[16 + wave] = s2; }
        __syncthreads();
        s1 += st_part[wave ^ 1];
        s2 += st_part[16 + (wave ^ 1)];
    }
    if (lane == 0 && run0 == 0) {
        const float m = s1 / (float)K;
        float var = s2 / (float)K - m * m;
        var = var > 0.f ? var : 0.f;
        st_mean[token] = pivot + m;
        st_rstd[token] = 1.0f / __builtin_sqrtf(var + a.eps);
    }
    __syncthreads();
    if (n >= a.N) return;
    float mean[8], rstd[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) { mean[e] = st_mean[tchunk * 8 + e]; rstd[e] = st_rstd[tchunk * 8 + e]; }
    const unsigned* xw = reinterpret_cast<const unsigned*>(xs) + tchunk * 8 * Q;
    for (int pass = 0;; ++pass) {
        const int kl = feature(pass);
        if (k0 + kl >= k1) break;
        unsigned x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = xw[e * Q + (kl >> 1)];
        const unsigned gn = gamma_of(k0 + feature(pass + 1)), bn = beta_of(k0 + feature(pass + 1));
        float g0, g1, b0, b1;
        ln_add_pair<BF>(gw, 0.f, g0, g1);
        ln_add_pair<BF>(bw, 0.f, b0, b1);
        ln_ushort8 o0, o1;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float lo, hi;
            ln_add_pair<BF>(x[e], -mean[e], lo, hi);
            o0[e] = ln_narrow<BF>(lo * rstd[e] * g0 + b0);
            o1[e] = ln_narrow<BF>(hi * rstd[e] * g1 + b1);
        }
        uint16_t* dst = a.out + (long)(k0 + kl) * a.ldo + n;
        ln_store<false>(dst, o0);
        ln_store<false>(dst + a.ldo, o1);
        gw = gn;
        bw = bn;
    }
}

}  // namespace
}  // namespace shflbw

extern "C" int shflbw_layernorm_transpose(const void* x, int64_t ldx, const void* gamma,
                                          const void* beta, float eps, int normalize, void* out,
                                          int64_t ldo, int64_t N, int K, shflbw_dtype dtype,
                                          void* stream)
{
    using namespace shflbw;
    if (dtype != SHFLBW_F16 && dtype != SHFLBW_BF16)
        return fail(SHFLBW_ERR_BAD_DTYPE, "dtype must be SHFLBW_F16 or SHFLBW_BF16");
    if (N < 0 || K <= 0) return fail(SHFLBW_ERR_BAD_SHAPE, "N < 0 or K <= 0");
    if (N == 0) return SHFLBW_OK;
    if (!x || !out) return fail(SHFLBW_ERR_NULL_ARG, "x and out must not be NULL");
    if (ldx < K || ldo < N) return fail(SHFLBW_ERR_BAD_SHAPE, "leading dimension too small");
    if (K % 8 || N % 8 || ldx % 8 || ldo % 8 || reinterpret_cast<uintptr_t>(x) % 16 ||
        reinterpret_cast<uintptr_t>(out) % 16 || (gamma && reinterpret_cast<uintptr_t>(gamma) % 16) ||
        (beta && reinterpret_cast<uintptr_t>(beta) % 16))
        return fail(SHFLBW_ERR_BAD_SHAPE,
                    "K, N and the leading dimensions must be multiples of 8 and all bases 16-byte aligned");
    if (normalize && !(eps >= 0.f)) return fail(SHFLBW_ERR_BAD_SHAPE, "eps must be >= 0");
    const int64_t wgs = (N + LN_TOK - 1) / LN_TOK;
    if (wgs > 0x7fffffffLL) return fail(SHFLBW_ERR_BAD_SHAPE, "grid too large");
    LnArgs a;
    a.x = static_cast<const uint16_t*>(x);
    a.gamma = static_cast<const uint16_t*>(gamma);
    a.beta = static_cast<const uint16_t*>(beta);
    a.out = static_cast<uint16_t*>(out);
    a.ldx = (long)ldx; a.ldo = (long)ldo; a.N = (long)N; a.K = K; a.eps = eps;
    a.normalize = normalize ? 1 : 0;
    a.stream = ((uintptr_t)(ldo * 2) | reinterpret_cast<uintptr_t>(out)) % 64 == 0;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const LnChoice choice = choose_layernorm(a.N, K, a.normalize != 0);
    if (choice.kernel == Ln::FEW) {
        const int few_tok = choice.tokens;
        LnFew f;
        f.blocks = (int)((N + few_tok - 1) / few_tok);
        int shares = (few_tok == 8 && f.blocks > 64 ? 256 : 128) / f.blocks;
        if (shares > K / 64) shares = K / 64;
        if (shares < 1) shares = 1;
        f.slice = ((K + shares - 1) / shares + 15) / 16 * 16;
        // (pitch / 2) mod 8, as in the LDS-resident kernel: 64 words of a read in 64 banks
        f.pitch = f.slice + (few_tok == 16 ? 8 : 0);
        f.total = f.blocks * ((K + f.slice - 1) / f.slice);
        f.per_xcd = (f.total + 7) / 8;
        const size_t bytes = (size_t)few_tok * f.pitch * 2 + 2 * few_tok * 4 + 2 * 16 * 4;
        typedef void (*few_fn)(LnArgs, LnFew);
        static const few_fn ftable[4] = {&layernorm_transpose_few_kernel<false, 16>, &layernorm_transpose_few_kernel<false, 8>,
                                         &layernorm_transpose_few_kernel<true, 16>, &layernorm_transpose_few_kernel<true, 8>};
        const int which = (dtype == SHFLBW_BF16 ? 2 : 0) + (few_tok == 8 ? 1 : 0);
        const few_fn fn = ftable[which];
        static thread_local int raised_few[4] = {-1, -1, -1, -1};
        int dev = 0;
        hipError_t ea = hipGetDevice(&dev);
        if (ea != hipSuccess) return fail(SHFLBW_ERR_HIP, "hipGetDevice: %s", hipGetErrorString(ea));
        if (raised_few[which] != dev) {
            ea = hipFuncSetAttribute(reinterpret_cast<const void*>(fn), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
            if (ea != hipSuccess) return fail(SHFLBW_ERR_HIP, "hipFuncSetAttribute: %s", hipGetErrorString(ea));
            raised_few[which] = dev;
        }
        hipLaunchKernelGGL(fn, dim3(8u * (unsigned)f.per_xcd), dim3(1024), bytes, st, a, f);
        hipError_t el = hipGetLastError();
        if (el != hipSuccess) return fail(SHFLBW_ERR_HIP, "kernel launch: %s", hipGetErrorString(el));
        return SHFLBW_OK;
    }
    if (choice.kernel == Ln::RESIDENT) {
        const int tok = choice.tokens;
        int pitch = 0;
        const size_t bytes = (size_t)ln_resident_bytes(tok, K, pitch);
        const int64_t rwgs = (N + tok - 1) / tok;
        if (rwgs > 0x7fffffffLL) return fail(SHFLBW_ERR_BAD_SHAPE, "grid too large");
        typedef void (*resident_fn)(LnArgs, int);
        static const resident_fn table[8] = {
            &layernorm_transpose_resident_kernel<false, 32, false>, &layernorm_transpose_resident_kernel<false, 32, true>,
            &layernorm_transpose_resident_kernel<false, 64, false>, &layernorm_transpose_resident_kernel<false, 64, true>,
            &layernorm_transpose_resident_kernel<true, 32, false>,  &layernorm_transpose_resident_kernel<true, 32, true>,
            &layernorm_transpose_resident_kernel<true, 64, false>,  &layernorm_transpose_resident_kernel<true, 64, true>};
        const int which = (dtype == SHFLBW_BF16 ? 4 : 0) + (tok == 64 ? 2 : 0) + (a.normalize ? 1 : 0);
        const resident_fn fn = table[which];
        // the attribute is raised once per kernel and device
        static thread_local int raised_on[8] = {-1, -1, -1, -1, -1, -1, -1, -1};
        int dev = 0;
        hipError_t ea = hipGetDevice(&dev);
        if (ea != hipSuccess) return fail(SHFLBW_ERR_HIP, "hipGetDevice: %s", hipGetErrorString(ea));
        if (raised_on[which] != dev) {
            ea = hipFuncSetAttribute(reinterpret_cast<const void*>(fn), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
            if (ea != hipSuccess) return fail(SHFLBW_ERR_HIP, "hipFuncSetAttribute: %s", hipGetErrorString(ea));
            raised_on[which] = dev;
        }
        hipLaunchKernelGGL(fn, dim3((unsigned)rwgs), dim3(1024), bytes, st, a, pitch);
        hipError_t el = hipGetLastError();
        if (el != hipSuccess) return fail(SHFLBW_ERR_HIP, "kernel launch: %s", hipGetErrorString(el));
        return SHFLBW_OK;
    }
    if (choice.kernel == Ln::REGISTER) {
        typedef void (*register_fn)(LnArgs);
#define SHFLBW_LN_REG(P, S) \
    &layernorm_transpose_register_kernel<false, false, P, S>, &layernorm_transpose_register_kernel<false, true, P, S>, \
    &layernorm_transpose_register_kernel<true, false, P, S>, &layernorm_transpose_register_kernel<true, true, P, S>
        static const register_fn rtable[32] = {SHFLBW_LN_REG(1, false), SHFLBW_LN_REG(2, false), SHFLBW_LN_REG(3, false),
                                               SHFLBW_LN_REG(4, false), SHFLBW_LN_REG(1, true),  SHFLBW_LN_REG(2, true),
                                               SHFLBW_LN_REG(3, true),  SHFLBW_LN_REG(4, true)};
#undef SHFLBW_LN_REG
        const int parts = (K + 4095) / 4096;
        const int64_t rwgs = (N + 31) / 32;
        if (rwgs > 0x7fffffffLL) return fail(SHFLBW_ERR_BAD_SHAPE, "grid too large");
        const int slices = (K + 1023) / 1024, shares = ln_register_shares(a.N, K, a.normalize != 0, a.stream != 0);
        a.slices_per_wg = (slices + shares - 1) / shares;
        const unsigned ry = (unsigned)((slices + a.slices_per_wg - 1) / a.slices_per_wg);
        const int which = (ry > 1 ? 16 : 0) + (parts - 1) * 4 + (dtype == SHFLBW_BF16 ? 2 : 0) + (a.normalize ? 1 : 0);
        const register_fn fn = rtable[which];
        const size_t bytes = (size_t)2 * 32 * (1024 + 4) * 2 + 2 * 32 * 4;
        static thread_local int raised_reg[32] = {-1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1,
                                                  -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1};
        int dev = 0;
        hipError_t ea = hipGetDevice(&dev);
        if (ea != hipSuccess) return fail(SHFLBW_ERR_HIP, "hipGetDevice: %s", hipGetErrorString(ea));
        if (raised_reg[which] != dev) {
            ea = hipFuncSetAttribute(reinterpret_cast<const void*>(fn), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
            if (ea != hipSuccess) return fail(SHFLBW_ERR_HIP, "hipFuncSetAttribute: %s", hipGetErrorString(ea));
            raised_reg[which] = dev;
        }
        hipLaunchKernelGGL(fn, dim3((unsigned)rwgs, ry), dim3(1024), bytes, st, a);
        hipError_t el = hipGetLastError();
        if (el != hipSuccess) return fail(SHFLBW_ERR_HIP, "kernel launch: %s", hipGetErrorString(el));
        return SHFLBW_OK;
    }
    // split the features over grid.y until there are about two workgroups per CU
    const int nblocks = (K + LN_FB - 1) / LN_FB;
    int split = 1;
    // every workgroup that shares a token block repeats the block's statistics sweep, so a
    // normalising launch stops splitting at one workgroup per CU
    while (wgs * split < (a.normalize ? 256 : 512) && split * 2 <= nblocks && split < 16) split *= 2;
    a.blocks_per_wg = (nblocks + split - 1) / split;
    const unsigned gy = (unsigned)((nblocks + a.blocks_per_wg - 1) / a.blocks_per_wg);
    const dim3 sgrid((unsigned)wgs, gy), sblock(64 * LN_WAVES);
    if (dtype == SHFLBW_BF16) {
        if (a.normalize) hipLaunchKernelGGL((layernorm_transpose_kernel<true, true>), sgrid, sblock, 0, st, a);
        else hipLaunchKernelGGL((layernorm_transpose_kernel<true, false>), sgrid, sblock, 0, st, a);
    } else {
        if (a.normalize) hipLaunchKernelGGL((layernorm_transpose_kernel<false, true>), sgrid, sblock, 0, st, a);
        else hipLaunchKernelGGL((layernorm_transpose_kernel<false, false>), sgrid, sblock, 0, st, a);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(SHFLBW_ERR_HIP, "kernel launch: %s", hipGetErrorString(e));
    return SHFLBW_OK;
}
