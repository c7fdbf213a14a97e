// Split form of the stage-sum linear layer (Eq. 20) for more than 16 tokens:
// Y[m][o] = sum_i X[m][i] W~[o][i] with the prefix weight
// W~ = sum over stages t < K of s_t (Q_t - z_t) formed once per tile in
// binary32 and split into three bfloat16 operands, so that a product takes
// three matrix-core passes whatever the stage count.
//
// Operands (v_mfma_f32_16x16x32_bf16, lane l: row / column n = l % 16,
// k-slice j = l / 16, a chunk = 128 inputs, lane j owning inputs
// 32 j .. 32 j + 31 of it, block b = inputs 32 j + 8 b .. + 7):
//   * B: W~'s 24 significant bits as three bfloat16, 8 bits each, by cutting
//     off: every product is exact and nothing of W~ is left out. A code needs
//     no conversion: masked in place it is the binary16 subnormal
//     Q 2^(p - 24), exact in v_fma_mix_f32, and s_t takes the factor
//     2^(24 - p);
//   * A: X as it is.
// bfloat16 has binary32's range, so a value's neighbours along its row, or in
// its tile, do not matter. Two binary16 operands and two passes took as long
// (the activations then need converting, with running bounds on the ranges of
// every token and row: 12288 x 4096, 2048 tokens, 4 / 3 stages 519 / 490
// against 519 / 496 us; 5120 x 5120, 48 tokens 43.2 against 30.9) and held 22
// bits of W~ at best, fewer the wider the ranges.
//
// Accumulation order: the chunks of a row in 4 contiguous quarters
// (ceil(chunks / 4) each), a quarter in stretches of 4 chunks, each
// accumulated from 0 in chunk order (block by block, the least operand
// first), and the stretches added in order. On rows of up to 2048 inputs a
// quarter is one stretch and the order does not depend on the tile shape or
// on which waves take the quarters: every token count gives the same results.
// On longer rows quarters of their own waves are summed before they meet.
//
// What bounds it: with many tokens the matrix cores are busy half of the time,
// and operand building, which two waves of a SIMD do not hide behind each
// other, takes the rest (12288 x 4096, 2048 tokens, 4 stages: 538 us, 383 TFLOP/s
// of the product, 1150 of the three passes; 777 us in the prefill form, which
// multiplies every stage's codes). Per chunk of 16 rows a wave forms its B
// operands with about 390 vector instructions at 4 stages (9 per element and
// 3.5 to split it) whatever the tokens; a SIMD spends 4 to 5 cycles on each and
// 10 issue cycles per MFMA, of 16 the MFMA takes. So the tile has as many tokens
// as registers and LDS allow (256: 16 accumulators and 16 running sums) before
// it has more rows. With few tokens the waves wait for their chunk's loads
// (5120 x 5120, 48 tokens: an instruction every 9 cycles and SIMD; 30.9 us,
// general kernel 56.6), and calls with few tiles rather split the quarters over
// waves than the tokens.
//
// Tried on the binary16 operands and not kept: 32 x 32 x 16 MFMAs with two of
// a SIMD's waves in alternate vector and matrix phases (562 us on the first
// shape above, no room for the quarters' running sums); the same phases with
// this tile, 64 inputs per step (638 us: twice the barriers and per-step
// work); operand building laid between the MFMAs of one wave by hand (822 us:
// one token tile in flight). With the three bfloat16: a sum for every stretch
// up to the end, so that rows of 8192 inputs too give the same results in
// every shape (registers spilled: 5120 x 5120, 48 tokens 33.9 -> 36.7 us).

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rrq_dma.h"
#include "rrq_launch.h"

namespace rrq_detail {
namespace {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

constexpr int kZpSymmetric = 2;
constexpr int kScaleF32 = 0, kScaleF16 = 1;
// Chunks accumulated before they are folded into the running sum. Error on
// random packages of 12288 x 4096, 2048 tokens, 4 stages / 5120 x 25600, 192 tokens, 1 stage and
// groups of 32, off 64 bits: 3.5e-7 / 4.5e-7 with 16 chunks, 3.5e-7 / 3.3e-7
// with 8, 2.6e-7 / 2.6e-7 with 4, for 516 / 336, 514 / 337 and 519 / 341 us.
constexpr uint32_t kFoldChunks = 4;

__device__ __forceinline__ f32x4 mfma(const u32x4 &a, const u32x4 &b, const f32x4 &c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                   __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// fma(s, half of q, c) with the low / high binary16 of q (subnormals kept).
__device__ __forceinline__ float fma_lo(float s, uint32_t q, float c)
{
    float d;
    asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel_hi:[0,1,0]" : "=v"(d) : "v"(s), "v"(q), "v"(c));
    return d;
}
__device__ __forceinline__ float fma_hi(float s, uint32_t q, float c)
{
    float d;
    asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel:[0,1,0] op_sel_hi:[0,1,0]"
        : "=v"(d) : "v"(s), "v"(q), "v"(c));
    return d;
}

// The bfloat16 pair of (a, b), cut off, and a and b less that (exact: what is
// left has the 16, then 8, lower significant bits). neg_lo and neg_hi hold
// the pairs (-1, 0) and (0, -1) in registers: written as a constant operand,
// -1 would be taken as a binary32.
__device__ __forceinline__ uint32_t cut_pair(float &a, float &b, uint32_t neg_lo, uint32_t neg_hi)
{
    const uint32_t h = __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302u);
    const bf16x2 hv = __builtin_bit_cast(bf16x2, h);
    a = __builtin_amdgcn_fdot2_f32_bf16(hv, __builtin_bit_cast(bf16x2, neg_lo), a, false);
    b = __builtin_amdgcn_fdot2_f32_bf16(hv, __builtin_bit_cast(bf16x2, neg_hi), b, false);
    return h;
}

// Scaling of a row's weights by a power of two where their magnitudes come
// near the ends of binary32's range, so that neither the scales' factors in
// dequant overflow nor the third operands underflow.
struct Range {
    float up, down;                      // applied to the scales, and to the sums
};
__device__ __forceinline__ Range range_of(int state)
{
    return state == 0 ? Range{1.0f, 1.0f} : state > 0 ? Range{0x1p-32f, 0x1p32f} : Range{0x1p64f, 0x1p-64f};
}

// A workgroup of WR x WQ waves owns 16 T tokens x 16 WR output rows: wave
// (wr, wq) rows 16 wr .. 16 wr + 15 for all the tokens, over every quarter of
// the chunks (WQ = 1) or over quarter wq (WQ = 4).
template <int K, int GPC, int WR, int WQ, int T>
struct Tile {
    static_assert(WQ == 1 || WQ == 4, "all quarters in turn, or one per wave");
    static_assert(T % WR == 0 || T < WR, "token tiles are prepared by the row waves");
    static constexpr int TOK = 16 * T;
    static constexpr int PT = T > WR ? T / WR : 1;           // token tiles a wave prepares
    static constexpr int X_DMA = 4 * PT;                     // 1 KiB loads per chunk
    // a wave's share of the package for one chunk: codes (stage t at 512 t,
    // row-major 16 x 32 bytes), scales and zero-points as 32-bit words
    // [stage][row][group of the chunk]
    static constexpr int CODE_DMA = (K + 1) / 2;
    static constexpr int PARAM_DMA = (K * 16 * GPC + 63) / 64;
    static constexpr int SCALES = CODE_DMA * 1024;
    static constexpr int ZEROS = SCALES + PARAM_DMA * 256;
    static constexpr int W_BYTES = ZEROS + PARAM_DMA * 256;
    static constexpr int W_DMA = CODE_DMA + 2 * PARAM_DMA;
    static constexpr int XB = TOK * 256;                     // per buffer and quarter
    static constexpr int W_BASE = 2 * WQ * XB;
    static constexpr int BYTES = W_BASE + WR * WQ * W_BYTES;
    static_assert(BYTES <= 160 * 1024, "LDS of a compute unit");
    static_assert(X_DMA + W_DMA <= 63, "vmcnt");
    static_assert(WQ == 1 || WR * WQ * T * 1024 <= W_BASE, "quarters meet in the X buffers");
};

template <int K, int GPC, int WR, int WQ, int T>
__global__ __launch_bounds__(64 * WR * WQ, WR * WQ >= 8 ? 2 : 1) void split_kernel(
    const uint32_t *__restrict__ codes, const char *__restrict__ scales,
    const float *__restrict__ zeros, int64_t rows, int64_t cols, int64_t plane_words,
    int64_t plane_groups, const uint16_t *__restrict__ X, int64_t n_tokens,
    float *__restrict__ Y, int zero_point, int scale_type, int row_pitch)
{
    using L = Tile<K, GPC, WR, WQ, T>;
    constexpr int G = 128 / GPC;
    __shared__ __attribute__((aligned(16))) char smem[L::BYTES];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wr = wave % WR, wq = wave / WR;
    const int n = lane & 15;            // A row (token of a tile), B column (row)
    const int j = lane >> 4;            // k-slice
    const bool sym = zero_point == kZpSymmetric;
    uint32_t neg_lo, neg_hi;
    asm volatile("s_mov_b32 %0, 0xbf80" : "=s"(neg_lo));
    asm volatile("s_mov_b32 %0, 0xbf800000" : "=s"(neg_hi));

    const int64_t m0 = (int64_t)(blockIdx.x / row_pitch) * L::TOK;
    const int64_t o_tile = (int64_t)(blockIdx.x % row_pitch) * (16 * WR), o0 = o_tile + 16 * wr;
    if (o_tile >= rows) return;         // (of the pitch only)
    const uint32_t tokens_here = (uint32_t)(n_tokens - m0 < L::TOK ? n_tokens - m0 : L::TOK);
    const int64_t rem = rows - o0;
    const uint32_t rows_here = rem <= 0 ? 0u : (uint32_t)(rem < 16 ? rem : 16);
    const uint32_t gpr = (uint32_t)(cols / G);
    const uint32_t row_bytes = (uint32_t)(cols / 4);
    const uint32_t x_row = (uint32_t)cols * 2;
    const uint32_t sbytes = scale_type == kScaleF32 ? 4 : 2;
    const uint32_t code_plane = (uint32_t)plane_words * 4;
    const uint32_t scale_plane = (uint32_t)plane_groups * sbytes;
    const uint32_t zero_plane = (uint32_t)plane_groups * 4;
    const int64_t o_first = rows_here ? o0 : 0;         // rows past the end read nothing
    const u32x4 dx = make_desc(X + m0 * cols, tokens_here * x_row);
    const u32x4 dc = make_desc(codes + o_first * (cols / 16),
                               rows_here ? (K - 1) * code_plane + rows_here * row_bytes : 0u);
    const u32x4 ds = make_desc(scales + o_first * gpr * sbytes,
                               rows_here ? (K - 1) * scale_plane + rows_here * gpr * sbytes : 0u);
    const u32x4 dz = make_desc(sym ? nullptr : zeros + o_first * gpr,
                               sym || !rows_here ? 0u : (K - 1) * zero_plane + rows_here * gpr * 4);

    const uint32_t chunks = (uint32_t)((cols + 127) / 128);
    const uint32_t per_q = (chunks + 3) / 4;
    // this wave's chunks: c_begin .. c_end - 1
    const uint32_t c_begin = WQ == 1 ? 0u : (per_q * wq < chunks ? per_q * wq : chunks);
    const uint32_t c_end = WQ == 1 ? chunks : (c_begin + per_q < chunks ? c_begin + per_q : chunks);
    const uint32_t steps = WQ == 1 ? chunks : per_q;

    // Activations: this wave stages and prepares token tiles t0 .. t0 + PT - 1
    // (none where the tiles are fewer than the waves). Slot s of a tile holds
    // token s / 16's piece (s % 16) ^ (token % 16); load i of a tile fills
    // tokens 4 i .. 4 i + 3. Tokens past the last lie past the descriptor and
    // read zeros.
    const int t0 = L::PT * wr;
    const bool stages_x = T >= WR || t0 < T;
    uint32_t dma_x[4], x_in[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t tok = (uint32_t)(4 * i + (lane >> 4));
        x_in[i] = 8u * ((uint32_t)n ^ tok);       // first input of the piece
        dma_x[i] = ((uint32_t)(16 * t0) + tok) * x_row + 2 * x_in[i];
    }
    // Codes: lane l fills bytes 16 (l % 2) of row (l % 32) / 2 in stage
    // 2 i + l / 32 (a stage past K - 1 is never used).
    const uint32_t dma_code = (uint32_t)((lane & 31) >> 1) * row_bytes + 16 * (uint32_t)(lane & 1) +
                              (uint32_t)(lane >> 5) * code_plane;
    uint32_t dma_par[L::PARAM_DMA], par_st[L::PARAM_DMA];
#pragma unroll
    for (int i = 0; i < L::PARAM_DMA; ++i) {
        const uint32_t s = (uint32_t)(i * 64 + lane);
        par_st[i] = s / (GPC * 16);
        dma_par[i] = ((s / GPC) % 16) * gpr + s % GPC;
    }
    const uint32_t lds0 = lds_address(&smem[0]);
    const uint32_t lds_w = lds0 + (uint32_t)(L::W_BASE + wave * L::W_BYTES);
    const char *my_w = smem + L::W_BASE + wave * L::W_BYTES;
    auto xbuf = [&](int b) { return smem + (b * WQ + wq) * L::XB; };

    auto issue_x = [&](uint32_t c, int b) {
        if (!stages_x) return;
        const uint32_t lds = lds0 + (uint32_t)(b * WQ + wq) * L::XB + (uint32_t)t0 * 4096;
#pragma unroll
        for (int i = 0; i < L::X_DMA; ++i) {
            uint32_t off = dma_x[i % 4];
            if (GPC > 1 && c * 128 + x_in[i % 4] >= (uint32_t)cols) off = kSkip;
            dma_x4(dx, c * 256 + (uint32_t)(i / 4) * 16 * x_row, lds + (uint32_t)i * 1024, off);
        }
    };
    auto issue_w = [&](uint32_t c) {
#pragma unroll
        for (int i = 0; i < L::CODE_DMA; ++i)
            dma_x4(dc, c * 32 + 2u * i * code_plane, lds_w + 1024u * i, dma_code);
#pragma unroll
        for (int i = 0; i < L::PARAM_DMA; ++i) {
            const bool in = par_st[i] < (uint32_t)K &&
                            (GPC == 1 || c * GPC + (uint32_t)(lane % GPC) < gpr);
            if (scale_type == kScaleF32)
                dma_dword(ds, c * (GPC * 4), lds_w + L::SCALES + 256u * i,
                          in ? dma_par[i] * 4 + par_st[i] * scale_plane : kSkip);
            else
                dma_ushort(ds, c * (GPC * 2), lds_w + L::SCALES + 256u * i,
                           in ? dma_par[i] * 2 + par_st[i] * scale_plane : kSkip);
            dma_dword(dz, c * (GPC * 4), lds_w + L::ZEROS + 256u * i,
                      in ? dma_par[i] * 4 + par_st[i] * zero_plane : kSkip);
        }
    };

    f32x4 acc[T], run[T];
#pragma unroll
    for (int q = 0; q < T; ++q) {
        acc[q] = (f32x4){0.f, 0.f, 0.f, 0.f};
        run[q] = acc[q];
    }

    // The lane's package words of one chunk: code words 2 j, 2 j + 1 of its
    // row, scales and zero-points of the group they lie in.
    u32x2 cw[K];
    uint32_t sw[K], zw[K];
    auto read_w = [&]() {
        const int gi = GPC == 1 ? 0 : j / (4 / GPC);
#pragma unroll
        for (int t = 0; t < K; ++t) {
            cw[t] = *reinterpret_cast<const u32x2 *>(my_w + 512 * t + 32 * n + 8 * j);
            const int e = 4 * ((16 * t + n) * GPC + gi);
            sw[t] = *reinterpret_cast<const uint32_t *>(my_w + L::SCALES + e);
            zw[t] = *reinterpret_cast<const uint32_t *>(my_w + L::ZEROS + e);
        }
    };
    // Adds the accumulators of the lanes with yes to their running sums.
    int state = 0;                      // of the lane's row: Range
    auto fold = [&](bool yes) {
        const float down = range_of(state).down;
#pragma unroll
        for (int q = 0; q < T; ++q)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                run[q][i] = yes ? run[q][i] + acc[q][i] * down : run[q][i];
                acc[q][i] = yes ? 0.0f : acc[q][i];
            }
    };
    auto fold_all = [&]() {
        if (__ballot(state != 0) != 0) {
            fold(true);
            return;
        }
#pragma unroll
        for (int q = 0; q < T; ++q) {
#pragma unroll
            for (int i = 0; i < 4; ++i) run[q][i] = run[q][i] + acc[q][i];
            acc[q] = (f32x4){0.f, 0.f, 0.f, 0.f};
        }
    };
    // Stage scales and zero terms of the lane's row for the chunk; if the
    // row's range changed, its accumulators are folded first.
    float sv[K][3], cz = 0.0f;
    auto params = [&]() {
        float s[K], z[K], m = 0.0f;
#pragma unroll
        for (int t = 0; t < K; ++t) {
            s[t] = scale_type == kScaleF32 ? __uint_as_float(sw[t])
                   : scale_type == kScaleF16
                       ? (float)__builtin_bit_cast(_Float16, (uint16_t)(sw[t] & 0xFFFFu))
                       : __uint_as_float(sw[t] << 16);
            z[t] = sym ? 2.0f : __uint_as_float(zw[t]);
            m = __builtin_fmaf(fabsf(s[t]), 3.0f + fabsf(z[t]), m);
        }
        // (bit patterns of non-negative floats compare like the floats)
        uint32_t e = __float_as_uint(m);
        const bool far = e != 0u && (e >= (223u << 23) || e < (63u << 23));
        if (__ballot(far || state != 0) != 0) {
            if constexpr (GPC >= 2) {
                const uint32_t o = (uint32_t)__shfl_xor((int)e, 32);
                e = e > o ? e : o;
            }
            if constexpr (GPC >= 4) {
                const uint32_t o = (uint32_t)__shfl_xor((int)e, 16);
                e = e > o ? e : o;
            }
            const int now = e == 0u ? state : e >= (223u << 23) ? 1 : e < (63u << 23) ? -1 : 0;
            fold(now != state);
            state = now;
        }
        const float up = range_of(state).up;
        float c = 0.0f;
#pragma unroll
        for (int t = 0; t < K; ++t) {
            const float ss = s[t] * up;
            c = __builtin_fmaf(-ss, z[t], c);
            sv[t][0] = ss * 0x1p20f;
            sv[t][1] = ss * 0x1p18f;
            sv[t][2] = ss * 0x1p16f;
        }
        cz = c;
    };

    // B operands of blocks 2 h, 2 h + 1 from the lane's code word h.
    u32x4 bw[3][2];
    auto dequant = [&](int h) {
        float w[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) w[e] = cz;
#pragma unroll
        for (int t = 0; t < K; ++t) {
            const uint32_t c = cw[t][h];
            const uint32_t up = c << 4, dn = c >> 6;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const uint32_t src = e < 2 ? up : e < 5 ? c : dn;
                const int v = e < 2 ? e : e < 5 ? e - 2 : e - 5;
                const uint32_t q = src & (0x00300030u << (2 * v));
                w[e] = fma_lo(sv[t][v], q, w[e]);
                w[e + 8] = fma_hi(sv[t][v], q, w[e + 8]);
            }
        }
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int p = 0; p < 3; ++p)
                    bw[p][b][v] = cut_pair(w[8 * b + 2 * v], w[8 * b + 2 * v + 1], neg_lo, neg_hi);
    };

    uint32_t q_left = per_q;            // chunks left in the quarter
    if (c_begin < c_end) {
        issue_w(c_begin);
        if (stages_x) {
            issue_x(c_begin, 0);
            wait_vm<0>();
        }
    }
    for (uint32_t it = 0; it < steps; ++it) {
        const uint32_t c = c_begin + it;
        const int b = (int)(it & 1);
        // every wave's activations of this chunk have landed, and every wave
        // is done with the other buffer
        __syncthreads();
        if (c >= c_end) continue;
        const bool last = q_left == 1 || c + 1 == c_end;   // of the quarter
        wait_vm<0>();                   // the package words have landed
        read_w();
        const char *lb = xbuf(b);
        params();
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            dequant(h);
            // The next chunk's loads go out between the products (its package
            // words into this one's place, which has been read). Loads past
            // the last chunk read other data or zeros, never used.
            if (h == 0) {
                issue_x(c + 1, b ^ 1);
            } else {
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                issue_w(c + 1);
            }
#pragma unroll
            for (int q = 0; q < T; ++q) {
                const char *xt = lb + (16 * q + n) * 256;
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const u32x4 a = *reinterpret_cast<const u32x4 *>(xt + 16 * ((4 * j + 2 * h + i) ^ n));
                    acc[q] = mfma(a, bw[2][i], acc[q]);
                    acc[q] = mfma(a, bw[1][i], acc[q]);
                    acc[q] = mfma(a, bw[0][i], acc[q]);
                }
            }
        }
        --q_left;
        // end of the quarter or of a stretch of it
        if (last || (per_q - q_left) % kFoldChunks == 0) fold_all();
        if (last) q_left = per_q;
        if (stages_x) wait_vm<L::W_DMA>();   // the next chunk's activations have landed
    }
    // no load may still write this workgroup's LDS once it ends or reuses it
    wait_vm<0>();

    if constexpr (WQ > 1) {
        // the quarters meet in LDS: tile q of wave v at (v T + q) KiB
        __syncthreads();
        f32x4 *red = reinterpret_cast<f32x4 *>(smem);
        if (wq > 0) {
#pragma unroll
            for (int q = 0; q < T; ++q) red[(wave * T + q) * 64 + lane] = run[q];
        }
        __syncthreads();
        if (wq > 0) return;
#pragma unroll
        for (int v = 1; v < WQ; ++v)
#pragma unroll
            for (int q = 0; q < T; ++q) {
                const f32x4 p = red[((v * WR + wr) * T + q) * 64 + lane];
#pragma unroll
                for (int i = 0; i < 4; ++i) run[q][i] = run[q][i] + p[i];
            }
    }
    // lane: tokens m0 + 16 q + 4 j + i of output row o0 + n
    if ((uint32_t)n < rows_here) {
#pragma unroll
        for (int q = 0; q < T; ++q)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t tk = (uint32_t)(16 * q + 4 * j + i);
                if (tk < tokens_here) Y[(m0 + tk) * rows + o0 + n] = run[q][i];
            }
    }
}

template <typename... Args>
hipError_t launch(void (*kernel)(Args...), int grid, int block, hipStream_t stream, Args... args)
{
    void *argv[] = {static_cast<void *>(&args)...};
    return hipLaunchKernel(reinterpret_cast<const void *>(kernel), dim3(grid), dim3(block),
                           argv, 0, stream);
}

// Tile shapes: A, B, C stage all quarters in turn (8 row waves, 256 / 128 /
// 64 tokens), D, E, F give each quarter its own waves (32 rows x 64 tokens,
// 32 x 32, 64 x 32), for calls with too few tiles to fill the chip. A compute
// unit runs one workgroup, or two of C and, at 1 and 2 stages, of E (LDS), so
// a call costs its rounds of workgroups times the shape's time per round, with
// one (kCost) or two (kPair) to a compute unit: in tenths of a microsecond per
// 4096 inputs by stages, measured with groups of 64 and 128 on 4096 to 16384
// rows at 64 to 2048 tokens, packages read from HBM.
enum Shape { A, B, C, D, E, F, kShapes };
constexpr int kRows[kShapes] = {128, 128, 128, 32, 32, 64};
constexpr int kTokens[kShapes] = {256, 128, 64, 64, 32, 32};
constexpr int kCost[4][kShapes] = {{1560, 900, 570, 205, 160, 240}, {1630, 970, 650, 230, 190, 280},
                                   {1720, 1060, 760, 260, 225, 340}, {1830, 1160, 860, 290, 265, 450}};
constexpr int kPair[4][kShapes] = {{0, 0, 1030, 0, 250, 0}, {0, 0, 1210, 0, 300, 0},
                                   {0, 0, 1360, 0, 0, 0}, {0, 0, 1540, 0, 0, 0}};

constexpr Shape shape_of(int wr, int t)
{
    return wr == 8 ? (t == 16 ? A : t == 8 ? B : C) : wr == 4 ? F : t == 4 ? D : E;
}

struct Call {
    const uint32_t *codes;
    const char *scales;
    const float *zeros;
    int64_t rows, cols;
    int k, zp, sdt;
    const uint16_t *X;
    int64_t n_tokens;
    float *Y;
    int cus;
    hipStream_t stream;
};

template <int K, int GPC, int WR, int WQ, int T>
hipError_t launch_t(const Call &c)
{
    // Workgroups go to the 8 XCDs in turn: with a pitch of a multiple of 8 the
    // token tiles of a row tile share an XCD, and its L2 the package's lines
    // (11000 x 4096, 2048 tokens, 4 stages 636 -> 503 us, 16000 x 5120, 100 tokens
    // 266 -> 117); not where the XCDs that get the rest would need another
    // round (10699 x 8192, 287 tokens 248 -> 402).
    const int64_t row_tiles = (c.rows + 16 * WR - 1) / (16 * WR);
    const int64_t token_tiles = (c.n_tokens + 16 * T - 1) / (16 * T);
    const int64_t tiles = row_tiles * token_tiles, per_xcd = (row_tiles + 7) / 8 * token_tiles;
    const int64_t slots = tiles > c.cus && kPair[K - 1][shape_of(WR, T)] ? 2 * c.cus : c.cus;
    const bool pitched = token_tiles > 1 &&
                         (per_xcd * 8 + slots - 1) / slots <= (tiles + slots - 1) / slots;
    const int row_pitch = (int)(pitched ? (row_tiles + 7) / 8 * 8 : row_tiles);
    const int grid = (int)(row_pitch * token_tiles);
    return launch(split_kernel<K, GPC, WR, WQ, T>, grid, 64 * WR * WQ, c.stream, c.codes,
                  c.scales, c.zeros, c.rows, c.cols, c.rows * c.cols / 16,
                  c.rows * c.cols * GPC / 128, c.X, c.n_tokens, c.Y, c.zp, c.sdt, row_pitch);
}

template <int GPC, int WR, int WQ, int T>
hipError_t launch_k(const Call &c)
{
    if constexpr (GPC > 1) {   // groups of 128 come with 3 or 4 stages only
        if (c.k == 1) return launch_t<1, GPC, WR, WQ, T>(c);
        if (c.k == 2) return launch_t<2, GPC, WR, WQ, T>(c);
    }
    switch (c.k) {
    case 3: return launch_t<3, GPC, WR, WQ, T>(c);
    case 4: return launch_t<4, GPC, WR, WQ, T>(c);
    default: return hipErrorInvalidValue;
    }
}

// A chunk takes 32 bytes of a row's line of codes and 4 to 16 of its lines of
// scales and zero-points, per stage, and the rows in flight hold theirs in the
// L2 (32 MB) until the next chunk. Where they outgrow it every chunk reads them
// again, which sets the time of C from about 36 MB of lines (one per row and
// stage and array) and, at 4 stages, of F past 16384 rows: 24 tokens, 4 stages,
// groups of 128 / 64, 24576 x 4096 C 110 / 116 us, 28672 x 4096 C 172 / 181, F 102 /
// 149, E 98 / 113. (Rows of up to 2048 inputs share their lines of scales:
// 24576 x 2048, 48 tokens, 4 stages C 47.5, D 50; with groups of 32 the other
// shapes lose as much.)
int64_t shape_cost(int s, int64_t rows, int64_t cols, int G, int k, int64_t n_tokens, int cus)
{
    const int64_t row_tiles = (rows + kRows[s] - 1) / kRows[s];
    const int64_t token_tiles = (n_tokens + kTokens[s] - 1) / kTokens[s];
    const int64_t tiles = row_tiles * token_tiles, left = tiles % (2 * cus);
    const int64_t one = kCost[k - 1][s], pair = kPair[k - 1][s];
    const int64_t c = pair == 0 ? (tiles + cus - 1) / cus * one
                                : tiles / (2 * cus) * pair + (left == 0 ? 0 : left <= cus ? one : pair);
    int64_t again = 0;
    if (cols > 2048 && G > 32 && s == C && (row_tiles < 2 * cus ? row_tiles : 2 * cus) * k > 732)
        again = rows * k * token_tiles * (G == 128 ? 125 : 150) / 10000;
    if (cols > 2048 && G > 32 && s == F && k == 4 && rows > 16384)
        again = rows * k * token_tiles * (G == 128 ? 85 : 120) / 10000;
    return c > again ? c : again;
}

// The cheapest shape and its cost (tenths of a microsecond per 4096 inputs).
Shape cheapest(int64_t rows, int64_t cols, int G, int k, int64_t n_tokens, int cus, int64_t *cost)
{
    Shape best = B;
    *cost = INT64_MAX;
    for (int s = kShapes - 1; s >= 0; --s) {
        const int64_t c = shape_cost(s, rows, cols, G, k, n_tokens, cus);
        if (c < *cost) {
            *cost = c;
            best = (Shape)s;
        }
    }
    return best;
}

template <int GPC>
hipError_t launch_g(const Call &c, Shape s)
{
    switch (s) {
    case A: return launch_k<GPC, 8, 1, 16>(c);
    case B: return launch_k<GPC, 8, 1, 8>(c);
    case C: return launch_k<GPC, 8, 1, 4>(c);
    case D: return launch_k<GPC, 2, 4, 4>(c);
    case E: return launch_k<GPC, 2, 4, 2>(c);
    case F: return launch_k<GPC, 4, 4, 2>(c);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

int split_shape(int64_t rows, int64_t cols, int G, int k, int64_t n_tokens, int cus,
                int64_t *cost)
{
    return cheapest(rows, cols, G, k, n_tokens, cus, cost);
}

int64_t split_cost(int64_t rows, int64_t cols, int G, int k, int64_t n_tokens, int cus)
{
    int64_t cost;
    const int shape = split_shape(rows, cols, G, k, n_tokens, cus, &cost);
    // The shapes with a quarter per wave read lines again as well, on 8193 to
    // 16384 rows from about 66 MB of lines (4 quarters' each), 50 MB on rows of
    // 8192 inputs or more; fitted, 24 tokens: 4 stages, groups of 128, 16384 x
    // 8192 171 us against 102 without it, 10922 x 12288 189 against 142, 16000 x
    // 6144 109 against 68; groups of 64, 10885 x 8192 161 against 90, 2 stages,
    // 16384 x 8192 125 against 56. (The general kernel takes 136, 147, 103, 137
    // and 91, the prefill form 101, 142 and 79. With smaller groups, 4 stages and
    // planes a multiple of an XCD's 4 MiB apart it loses as much: 16384 x 8192,
    // groups of 64, 286 against 250.)
    const bool aliased = G < 128 && k == 4 && rows * cols % (1 << 24) == 0;
    if (shape >= D && (rows > 8192 || (rows == 8192 && cols >= 12288)) && rows <= 16384 &&
        rows * k > (cols < 8192 ? 43000 : 32600) && !aliased) {
        const int64_t token_tiles = (n_tokens + kTokens[shape] - 1) / kTokens[shape];
        const int64_t again = rows * k * (75 + cols / 192) * (G == 128 ? 10 : 14) / 100000 * token_tiles;
        if (again > cost) cost = again;
    }
    return cost;
}

bool linear_split_fits(int64_t rows, int64_t cols, int G, int k, int64_t n_tokens, int cus)
{
    // The activation descriptor spans at most 256 rows of X (under 2^31
    // bytes), and the grid fits an int.
    const int64_t tiles32 = ((rows + 31) / 32 + 7) * ((n_tokens + 31) / 32);
    if (n_tokens <= 16 || cols > 65536 || tiles32 >= (1ll << 31)) return false;
    if (G == 128) {
        if (n_tokens < kPrefillMinTokens && linear_prefill_fits(rows, cols, G, k, n_tokens, cus))
            return false;
        // One and two stages stay with the forms that multiply the stages'
        // codes: no more passes than three, and no operand arithmetic. (Ahead
        // from 128 x 128 tiles on: 12288 x 4096, 128 tokens, 2 stages 55
        // against 63 us. With few tiles this form would be: 4096 x 4096, 64 /
        // 128 tokens, 2 stages 19 / 23 against 23 / 37.)
        if (k < 3) return false;
        // Against the prefill form: ahead once the 128 x 128 tiles (B) give
        // nearly every compute unit one. 4 / 3 stages: 4096 x 4096, 1024
        // tokens 114 / 107 against 142 / 110 us, 12288 x 4096, 500 tokens 163
        // / 153 against 257 / 201, 2048 tokens 519 / 496 against 769 / 656;
        // with half as many tiles (4096 x 4096, 500 tokens) 88 / 79 against
        // 86 / 71.
        if (n_tokens >= kPrefillMinTokens) {
            const int64_t tiles = ((rows + 127) / 128) * ((n_tokens + 127) / 128);
            return 8 * tiles >= (k == 4 ? 7 : 8) * (int64_t)cus;
        }
    }
    return split_cost(rows, cols, G, k, n_tokens, cus) < general_cost(rows, n_tokens, G, k, cus);
}

hipError_t launch_linear_split(const uint32_t *codes, const void *scales, const float *zeros,
                               int64_t rows, int64_t cols, int G, int k, int zero_point,
                               int scale_type, const uint16_t *X, int64_t n_tokens, float *Y,
                               int cus, hipStream_t stream)
{
    const Call c = {codes, static_cast<const char *>(scales), zeros, rows, cols, k, zero_point,
                    scale_type, X, n_tokens, Y, cus, stream};
    int64_t cost;
    const Shape shape = cheapest(rows, cols, G, k, n_tokens, cus, &cost);
    switch (G) {
    case 32: return launch_g<4>(c, shape);
    case 64: return launch_g<2>(c, shape);
    case 128: return launch_g<1>(c, shape);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace rrq_detail
