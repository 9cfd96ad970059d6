// Many-token kernel of the residual-binary layer: a matrix-core GEMM, one launch, no pre-pass.
//
// Section 4.1 / Eq. (stacked binary weight): Y[t][i] = sum_k g_k[i] * sum_j B_k[i][j] * (h_k[j] X[t][j]).
// With dozens of tokens per weight and more this is a dense contraction Y = W_hat X with
// W_hat = sum_k g_k (.) B_k (.) h_k (Alg. 2, "compute layer output") on v_mfma_f32_32x32x16_f16.  The left
// operand is W_hat itself, built in registers from the packed signs on the way to the matrix
// instruction and never stored.  Per pair of fp16 elements: a 64-bit shift brings the two sign bits of two paths
// to bits 15 and 31 of their words (with a shift per path 4096 x 4096 at 333 tokens took 29.7 us where this took 28.5, three paths 28672 x 8192 at 512 288 and
// 276), one three-input logic operation per path puts them on the pair of h_k.  Two forms add the paths up:
//   * h_0 B_0 + rho_k h_k B_k with rho_k = g_k / g_0 in fp16 and g_0 on the fp32 sums at the end, a packed fused multiply-add per
//     path but the first: four vector instructions for two paths, one rounding of the sum and one of rho_k.  Taken by a workgroup in all of
//     whose rows path 0 weighs (g_k^2 |h_k|^2) as much as the others together, as it does in a layer whose paths are residuals of one another:
//     there the rounding of rho_k, relative to the row, is no larger than that of g_0 h_0 B_0 which it replaces;
//   * G_k h_k B_k summed over all paths, G_k = g_k but for a power of two per row, exact: a multiplication more and a wait state for its
//     result, six issue slots per pair against four, and a rounding per path.
// Measured, first form and second: 4096 x 11008 at 512 tokens 70 and 76 us, 28672 x 8192 at 100 79 and 82, at 2048 937 and 976; three
// paths, 11008 x 4096 at 2048 224 and 235.  Error against fp64, all rows and the worst of 256: even scales (residual paths) 2.0e-4 and 2.6e-4
// (2.7e-4 and 4.6e-4 in the second form), scales spread by e^N(0,1) 2.8e-4 and 3.4e-4 in the second (2.3e-4 and 4.9e-4 in the first; and a
// per cent where an uneven h_1 stands beside a row without g_0).  Powers of two (s_k that brings max|h_k| into [1/4, 1/2)) keep the
// terms in fp16's normal range however the layer splits its magnitude.
//
// What bounds it: the vector instructions that build W_hat, until some 128 tokens share them, then the
// matrix units (a wavefront hides about six vector instructions behind one 32x32x16 instruction,
// measured; the rest add up).  So a workgroup (8 wavefronts, one workgroup per compute unit) takes as
// many tokens as still leave one workgroup per compute unit:
//   * a wavefront owns 64 rows and all 32 NT tokens of the workgroup, so no two wavefronts build the same
//     piece of W_hat for the same tokens; WR wavefronts stand side by side along the rows, and
//     WK = 8 / WR groups of them share out the columns and add their sums in LDS at the end;
//   * a step is 128 columns per group.  X goes through LDS (two buffers): whole 256-byte rows are
//     fetched, converted if they are bfloat16, and stored as pairs (e, e + 4) of eight columns, the
//     order in which one shift of a native sign word serves both halves of a register.  The scales h are
//     K more rows of the same slab.  A part of a slab is requested a whole step before it is
//     written, in two places of the step, so that the requests of eight wavefronts do not queue up;
//   * sign words come straight from memory into the lane that needs them (lane (r, kg) takes columns 64 kg ..
//     of the step): no lane exchange;
//   * the tile is brought to the output's type in LDS and stored as whole rows;
//   * the left operand of the next row block is built between the matrix instructions of this one.
//
// Measured, fp16, two paths, first form, calls in a row in a graph, from card to card and with cold clocks: 4096 x 4096 at 333 tokens 23-28 us,
// 11008 x 4096 45-52 us, 4096 x 11008 54-63 us, 8192 x 8192 at 1024 134-145 us (1.0 PFLOP/s), 28672 x 8192 at 2048 tokens 0.92-0.97 ms (1.07 among
// other work), where the power that the matrix units may draw is the bound: the same call on activations of zero takes 0.71 ms (torch's product of fp16 matrices 0.82 and 0.66).
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>

#include <algorithm>
#include <atomic>
#include <type_traits>

#include "rabit.h"
#include "rb_device.h"
#include "rb_internal.h"
#include "rb_layout.h"
#include "rb_mx_device.h"

namespace rb {
namespace gemm {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef _Float16 v2h __attribute__((ext_vector_type(2)));
typedef float v2f __attribute__((ext_vector_type(2)));

constexpr int WAVES = 8, MB = 2;                 // wavefronts of a workgroup, blocks of 32 rows of a wavefront
constexpr int STEP_COLS = 128, ROW_BYTES = 256;  // columns of a step; a token's fp16 values of them
constexpr int MAX_IN = 1 << 22;                  // 32-bit offsets into the rows of a tile

template <int K, int NT> __host__ __device__ constexpr int slab_bytes() { return (32 * NT + K) * ROW_BYTES; }
template <int K, int NT, int WR> __host__ __device__ constexpr int lds_bytes() { return 2 * (WAVES / WR) * slab_bytes<K, NT>(); }

struct Args {
    const uint32_t *bits;
    const __half *g, *h;
    const void *X;
    void *Y;
    int out, in, T, out_dtype;
};

__device__ __forceinline__ uint32_t pack_halves(_Float16 lo, _Float16 hi)
{
    return (uint32_t)__builtin_bit_cast(unsigned short, lo) | ((uint32_t)__builtin_bit_cast(unsigned short, hi) << 16);
}
// eight values in memory order as the pairs (e, e + 4), e = 0..3: the order in which two shifts of a
// native sign word by 4 e bring the bits of a pair to bits 15 and 31
__device__ __forceinline__ uint4 pair_order(uint4 v)
{
    return make_uint4(__builtin_amdgcn_perm(v.z, v.x, 0x05040100u), __builtin_amdgcn_perm(v.z, v.x, 0x07060302u),
                      __builtin_amdgcn_perm(v.w, v.y, 0x05040100u), __builtin_amdgcn_perm(v.w, v.y, 0x07060302u));
}
// (as vectors of two: one conversion instruction per pair)
__device__ __forceinline__ uint32_t low_bf16(uint32_t a, uint32_t b)
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((v2f){__uint_as_float(a << 16), __uint_as_float(b << 16)}, v2h));
}
__device__ __forceinline__ uint32_t high_bf16(uint32_t a, uint32_t b)
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((v2f){__uint_as_float(a & 0xffff0000u), __uint_as_float(b & 0xffff0000u)}, v2h));
}
__device__ __forceinline__ uint4 pair_order_of_bf16(uint4 v)
{
    return make_uint4(low_bf16(v.x, v.z), high_bf16(v.x, v.z), low_bf16(v.y, v.w), high_bf16(v.y, v.w));
}
// of eight fp16 values
__device__ __forceinline__ void largest_and_squares(uint4 v, float &m, float &sq)
{
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const v2h p = __builtin_bit_cast(v2h, w[i]);
        m = fmaxf(m, fmaxf(fabsf((float)p[0]), fabsf((float)p[1])));
        sq = __builtin_amdgcn_fdot2(p, p, sq, false);
    }
}
// all lanes' values combined, left in every lane (every lane must be active): data-parallel moves inside a row of 16 lanes, register
// swaps beyond; by lane exchanges through LDS the two reductions took 0.4 us of a call
template <typename F> __device__ __forceinline__ float over_wave(float v, F op)
{
    v = op(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xf, 0xf, false)));      // quad_perm [1,0,3,2]
    v = op(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xf, 0xf, false)));      // quad_perm [2,3,0,1]
    v = op(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x141, 0xf, 0xf, false)));     // row_half_mirror
    v = op(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x140, 0xf, 0xf, false)));     // row_mirror
    const auto rows = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = op(__uint_as_float(rows[0]), __uint_as_float(rows[1]));
    const auto halves = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return op(__uint_as_float(halves[0]), __uint_as_float(halves[1]));
}
// loads that return zero past the end of their buffer (NOWHERE always is)
constexpr uint32_t NOWHERE = 0x40000000u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer(const void *p, size_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ uint4 buffer_load(__amdgpu_buffer_rsrc_t rs, uint32_t lane_offset, int offset)
{
    return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)lane_offset, offset, 0));
}

// K paths, NT groups of 32 tokens, WR wavefronts along the rows (the other WAVES / WR share out the columns);
// BF16: X is bfloat16.  h starts at a multiple of 16 bytes (its rows then do too).  14 words of single arguments, which the compiler has put
// into registers at the start (build.py asks for it; two 7B-shaped blocks at 333 tokens 567 us with the arguments in memory, 560 so)
template <int K, int NT, int WR, bool BF16>
__global__ __launch_bounds__(WAVES * 64, 1) void gemm_kernel(Address bits_, Address h_, Address X_, Address g_, Address Y_, int out, int in, int T, int out_dtype)
{
    const uint32_t *const bits = global_at<const uint32_t>(bits_);
    const __half *const h = global_at<const __half>(h_), *const g = global_at<const __half>(g_);
    const uint8_t *const X = global_at<const uint8_t>(X_);
    uint8_t *const Y = global_at<uint8_t>(Y_);
    constexpr int WK = WAVES / WR, GT = 64 * WR;               // column groups; threads of one
    constexpr int TOK = 32 * NT, XL = TOK * 16 / GT, XP = XL / 2;     // tokens of a tile; 16-byte loads of X per thread and step, in two parts
    constexpr int SLAB = slab_bytes<K, NT>();
    static_assert(MB == 2 && TOK * 16 % GT == 0 && XL % 2 == 0, "whole loads per thread");
    static_assert(TOK * (64 * WR * 4 + 16) <= lds_bytes<K, NT, WR>() && 32768 * NT <= lds_bytes<K, NT, WR>(), "what reuses the slabs fits");
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];       // [column group][2][SLAB]
    __shared__ float red[2 * RB_MAX_K][WAVES];
    __shared__ __attribute__((aligned(16))) float row_scale[64 * WR];
    __shared__ int uneven[WR];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = wave / WR, wr = wave % WR;
    const int r = lane & 31, kg = lane >> 5;
    const int RT = row_tiles(out), CT = col_tiles(in);
    const int TB = (T + TOK - 1) / TOK, RB = (RT + 2 * MB * WR - 1) / (2 * MB * WR);
    // workgroups go round the eight XCDs: each takes a run of tiles, token blocks fastest, so its L2 sees
    // an eighth of the signs and all of X
    const int tiles = RB * TB, per = (tiles + 7) / 8, id = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per || id >= tiles) return;
    const int t0 = id % TB * TOK, rt0 = (id / TB * WR + wr) * 2 * MB;

    // steps of 128 columns, a run of them per column group
    const int n128 = (in + STEP_COLS - 1) / STEP_COLS;
    const int s_begin = n128 * grp / WK, s_end = n128 * (grp + 1) / WK, rounds = (n128 + WK - 1) / WK;

    // ---- staging: thread gid of a column group takes chunk gid % 16 (8 columns) of rows gid / 16 + ..
    // Everything a step advances is uniform over the wavefront; a lane keeps 32-bit offsets
    const int gid = tid - grp * GT, ch = gid & 15, row0 = gid >> 4;
    uint8_t *const slab0 = lds + (size_t)grp * 2 * SLAB;
    const uint8_t *const Xt = X + (size_t)t0 * in * 2;
    uint32_t x_off[XL];
#pragma unroll
    for (int i = 0; i < XL; ++i) x_off[i] = (uint32_t)min(row0 + i * (GT / 16), T - 1 - t0) * (uint32_t)in * 2u + (uint32_t)ch * 16u;
    const uint32_t h_off = row0 < K ? ((uint32_t)row0 * (uint32_t)in + (uint32_t)ch * 8u) * 2u : NOWHERE;
    const __amdgpu_buffer_rsrc_t x_rs = buffer(Xt, (size_t)min(TOK, T - t0) * in * 2), h_rs = buffer(h, (size_t)K * in * 2);
    constexpr bool SHORT = NT == 4;                            // registers for half of a slab only
    uint4 xs[SHORT ? XP : XL], hs;
    auto reg = [&](int i) { return SHORT ? i % XP : i; };
    // (no branch: the waits further down count the loads that came after)
    auto request = [&](int s, int part) {
        const bool real = s < s_end && s * STEP_COLS + ch * 8 < in;        // columns past the end read as zero
        const int at = min(s, n128 - 1) * ROW_BYTES;
#pragma unroll
        for (int i = part * XP; i < part * XP + XP; ++i) xs[reg(i)] = buffer_load(x_rs, real ? x_off[i] : NOWHERE, at);
        if (part == 0) hs = buffer_load(h_rs, real ? h_off : NOWHERE, at);
    };
    float h_scale = 1.f;
    // a chunk sits at position chunk ^ (row % 16) of its row: neither these writes nor the operand reads collide on LDS banks
    auto put = [&](int buf, int part) {
        uint8_t *const dst = slab0 + buf * SLAB;
#pragma unroll
        for (int i = part * XP; i < part * XP + XP; ++i) {
            const int row = row0 + i * (GT / 16);
            *reinterpret_cast<uint4 *>(dst + row * ROW_BYTES + ((ch ^ (row & 15)) * 16)) = BF16 ? pair_order_of_bf16(xs[reg(i)]) : pair_order(xs[reg(i)]);
        }
        if (part == 0 && row0 < K) {
            uint4 v = hs;
            uint32_t *const w = reinterpret_cast<uint32_t *>(&v);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const v2h p = __builtin_bit_cast(v2h, w[i]);
                w[i] = pack_halves((_Float16)((float)p[0] * h_scale), (_Float16)((float)p[1] * h_scale));
            }
            *reinterpret_cast<uint4 *>(dst + (TOK + row0) * ROW_BYTES + ch * 16) = pair_order(v);
        }
    };
    // sign words of row block b: lane (r, kg) holds, for row r of the 32, columns 64 kg + 32 u .. of the step
    // (the words of paths 0 and 1 in one register pair: they share their shifts)
    struct Words { unsigned long long pair; uint32_t third; };
    Words w[MB][2], wn[MB][2];
    uint32_t w_off[MB];
    const int rt_safe = min(rt0, RT - 1);
    const uint8_t *const tile_bits = reinterpret_cast<const uint8_t *>(bits + (size_t)rt_safe * CT * tile_words(K));
#pragma unroll
    for (int b = 0; b < MB; ++b) {
        const uint32_t rt = (uint32_t)(min(rt0 + 2 * b + (r >> 4), RT - 1) - rt_safe);      // row tiles past the end: the last one, not stored
        w_off[b] = (rt * (uint32_t)CT * tile_words(K) + ((uint32_t)(r & 15) + 32u * kg) * (2 * K)) * 4u;
    }
    auto load_words = [&](int s, Words (&to)[MB][2]) {
        const int sc = min(s, n128 - 1);
        const uint8_t *const p = tile_bits + (size_t)(sc >> 1) * (tile_words(K) * 4) + (sc & 1) * (4 * K);
#pragma unroll
        for (int b = 0; b < MB; ++b)
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const uint8_t *const at = p + w_off[b] + u * (16 * 2 * K * 4);
                uint32_t v[K];
#pragma unroll
                for (int k = 0; k < K; ++k) v[k] = *reinterpret_cast<const uint32_t *>(at + k * 4);
                to[b][u].pair = (unsigned long long)v[1] << 32 | v[0];
                if (K == 3) to[b][u].third = v[K - 1];
            }
    };
    request(s_begin, 0);
    if (!SHORT) request(s_begin, 1);
    load_words(s_begin, w);
    float gv[MB][K];
#pragma unroll
    for (int b = 0; b < MB; ++b)
#pragma unroll
        for (int k = 0; k < K; ++k) gv[b][k] = __half2float(g[(size_t)k * out + min(rt0 * TILE_ROWS + 32 * b + r, out - 1)]);

    // ---- powers of two that bring the scales h of a path to [1/4, 1/2), and the sum of their squares
    float mx_h[K], sq_h[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        mx_h[k] = sq_h[k] = 0.f;
        for (int j = tid * 8; j < in; j += WAVES * 64 * 8) largest_and_squares(buffer_load(h_rs, (uint32_t)(k * in + j) * 2u, 0), mx_h[k], sq_h[k]);
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
        mx_h[k] = over_wave(mx_h[k], [](float a, float b) { return fmaxf(a, b); });
        sq_h[k] = over_wave(sq_h[k], [](float a, float b) { return a + b; });
        if (lane == 0) { red[2 * k][wave] = mx_h[k]; red[2 * k + 1][wave] = sq_h[k]; }
    }
    __syncthreads();
    float sk[K], weight[MB][K];                                // weight: what path k adds to the squared norm of a row of W_hat
#pragma unroll
    for (int k = 0; k < K; ++k) {
        float a = 0.f, sq = 0.f;
#pragma unroll
        for (int v = 0; v < WAVES; ++v) { a = fmaxf(a, red[2 * k][v]); sq += red[2 * k + 1][v]; }
        sk[k] = mx::input_scale(a);
        if (row0 == k) h_scale = sk[k];
#pragma unroll
        for (int b = 0; b < MB; ++b) {
            weight[b][k] = gv[b][k] * gv[b][k] * sq;
            gv[b][k] = a > 0.f ? gv[b][k] / sk[k] : 0.f;       // (a path without a scale has no say)
        }
    }
    // ---- may path 0 carry the others (the first form above)?  (a NaN compares false: no)
    bool carries = true;
#pragma unroll
    for (int b = 0; b < MB; ++b) {
        float others = 0.f;
#pragma unroll
        for (int k = 1; k < K; ++k) others += weight[b][k];
        carries = carries && others <= weight[b][0];
    }
    const bool all_carry = __all(carries);
    if (grp == 0 && lane == 0) uneven[wr] = !all_carry;
    // ---- a row of W_hat as base (h_0 B_0 + sum_k rho_k h_k B_k), base = g_0, if so; else (further down) as base (sum_k G_k h_k B_k), base a
    // power of two that leaves the row's largest G_k in [1/4, 1/2)
    auto both = [](float f) { const _Float16 v = (_Float16)f; return (v2h){v, v}; };
    v2h coef[MB][K];
#pragma unroll
    for (int b = 0; b < MB; ++b) {
        coef[b][0] = both(1.f);
#pragma unroll
        for (int k = 1; k < K; ++k) coef[b][k] = both(gv[b][0] != 0.f ? gv[b][k] / gv[b][0] : 0.f);
        if (grp == 0 && kg == 0) row_scale[64 * wr + 32 * b + r] = gv[b][0];
    }
    put(0, 0);
    if (SHORT) request(s_begin, 1); else request(s_begin + 1, 0);
    put(0, 1);
    if (!SHORT) request(s_begin + 1, 1);
    __syncthreads();
    bool ratios = true;                                        // uniform over the workgroup
#pragma unroll
    for (int v = 0; v < WR; ++v) ratios = ratios && __builtin_amdgcn_readfirstlane(uneven[v]) == 0;
    if (!ratios)
#pragma unroll
        for (int b = 0; b < MB; ++b) {
            float most = fabsf(gv[b][0]);
#pragma unroll
            for (int k = 1; k < K; ++k) most = fmaxf(most, fabsf(gv[b][k]));
            const float S = mx::input_scale(most);
#pragma unroll
            for (int k = 0; k < K; ++k) coef[b][k] = both(gv[b][k] * S);
            if (grp == 0 && kg == 0) row_scale[64 * wr + 32 * b + r] = 1.f / S;
        }

    v16f acc[MB][NT];
#pragma unroll
    for (int b = 0; b < MB; ++b)
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[b][n][e] = 0.f;

    // chunk 8 kg + 4 u + c of a row is columns 64 kg + 32 u + 8 c ..
    const int x_addr = r * ROW_BYTES + (((8 * kg) ^ (r & 15)) * 16), h_addr = TOK * ROW_BYTES + 8 * kg * 16;
    constexpr int XB = NT <= 3 ? 2 : 1;                        // operands of X read one contraction ahead (registers)
    v8h x[XB][NT];
    uint4 hv[2][K];
    auto fetch_h = [&](const uint8_t *slab, int uc, int to) {
#pragma unroll
        for (int k = 0; k < K; ++k) hv[to][k] = *reinterpret_cast<const uint4 *>(slab + h_addr + k * ROW_BYTES + uc * 16);
    };
    auto fetch_x = [&](const uint8_t *slab, int uc, int to) {
#pragma unroll
        for (int n = 0; n < NT; ++n) x[to][n] = *reinterpret_cast<const v8h *>(slab + (x_addr ^ (uc * 16)) + n * 32 * ROW_BYTES);
    };
    // register j of the left operand of row block b, columns of contraction uc: W_hat of a pair of columns
    auto expand = [&](auto by_ratios, uint4 &a, int b, int uc, int from, int j) {
        v2h sum;
        uint32_t at_top[3];
        shift_left(w[b][uc >> 2].pair, 15 - 4 * j - (uc & 3), at_top[0], at_top[1]);
        if (K == 3) at_top[2] = w[b][uc >> 2].third << (15 - 4 * j - (uc & 3));
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const uint32_t hw = reinterpret_cast<const uint32_t *>(&hv[from][k])[j];
            const v2h v = __builtin_bit_cast(v2h, hw ^ (at_top[k] & 0x80008000u));
            if (k == 0) sum = decltype(by_ratios)::value ? v : coef[b][0] * v;
            else sum = __builtin_elementwise_fma(coef[b][k], v, sum);
        }
        reinterpret_cast<uint32_t *>(&a)[j] = __builtin_bit_cast(uint32_t, sum);
    };
    auto contract = [&](auto by_ratios, int from, int to) {
        for (int i = from; i < to; ++i) {
            const int s = s_begin + i;
            const uint8_t *const slab = slab0 + (i & 1) * SLAB;
            fetch_h(slab, 0, 0);
            fetch_x(slab, 0, 0);
            uint4 a[2];
#pragma unroll
            for (int j = 0; j < 4; ++j) expand(by_ratios, a[0], 0, 0, 0, j);
#pragma unroll
            for (int uc = 0; uc < 8; ++uc) {
                const int at = uc & 1;
                // the next step's slab is written part by part.  Each part's registers are asked for again at once (a
                // step later they are needed), or half a step before they are needed
                if (SHORT) {
                    if (uc == 0) request(s + 1, 0);
                    if (uc == 4) { put((i + 1) & 1, 0); request(s + 1, 1); }
                } else {
                    if (uc == 1) { put((i + 1) & 1, 0); request(s + 2, 0); }
                    if (uc == 5) { put((i + 1) & 1, 1); request(s + 2, 1); }
                }
                if (uc == 3) load_words(s + 1, wn);
                if (uc < 7) fetch_h(slab, uc + 1, at ^ 1);
                if (uc < 7 && XB == 2) fetch_x(slab, uc + 1, at ^ 1);
                if (uc > 0 && XB == 1) fetch_x(slab, uc, 0);
                __builtin_amdgcn_sched_barrier(0);
                // between the matrix instructions of one row block: the left operand of the next
#pragma unroll
                for (int b = 0; b < MB; ++b) {
                    const int next_uc = b + 1 < MB ? uc : uc + 1, next_b = (b + 1) % MB;
#pragma unroll
                    for (int n = 0; n < NT; ++n) {
                        acc[b][n] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, a[b & 1]), x[at % XB][n], acc[b][n], 0, 0, 0);
                        if (next_uc < 8)
#pragma unroll
                            for (int j = 4 * n / NT; j < 4 * (n + 1) / NT; ++j) expand(by_ratios, a[(b + 1) & 1], next_b, next_uc, next_uc & 1, j);
                        if (NT > 2) __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
            if (SHORT) put((i + 1) & 1, 1);
#pragma unroll
            for (int b = 0; b < MB; ++b)
#pragma unroll
                for (int u = 0; u < 2; ++u) w[b][u] = wn[b][u];
            __syncthreads();
        }
    };
    // (one after the other, so that the second takes over the registers of the first; as the two sides of a branch they were kept
    // twice and spilled up to 21)
    const int by_ratios = ratios ? rounds : 0;
    contract(std::true_type(), 0, by_ratios);
    contract(std::false_type(), by_ratios, rounds);

    // ---- sums of the column groups.  The tile is MB x NT x 4 pieces of four registers; each group adds up the pieces of an equal share
    // of it and hands the others theirs, so all wavefronts write, read and (below) convert (the upper half handing everything to the lower, twice with four
    // groups: 4096 x 4096 at 333 tokens 25.0 us)
    constexpr int PIECES_ALL = MB * NT * 4, SHARE = PIECES_ALL / WK;
    static_assert(WK == 2 || WK == 4, "`sum` below adds two or four");
    static_assert(PIECES_ALL % WK == 0 && (WK - 1) * WR * PIECES_ALL * 1024 <= lds_bytes<K, NT, WR>(), "equal shares, room for them");
    float4 *const part = reinterpret_cast<float4 *>(lds);
    auto piece = [&](int f) { return acc[f / (NT * 4)][f / 4 % NT]; };
    auto at = [&](int owner, int from, int f) { return part + ((((owner * (WK - 1) + (from < owner ? from : from - 1)) * WR + wr) * SHARE + f % SHARE) * 64 + lane); };
#pragma unroll
    for (int o = 0; o < WK; ++o)
        if (grp != o)
#pragma unroll
            for (int f = o * SHARE; f < (o + 1) * SHARE; ++f) {
                const v16f v = piece(f);
                *at(o, grp, f) = make_float4(v[f % 4 * 4], v[f % 4 * 4 + 1], v[f % 4 * 4 + 2], v[f % 4 * 4 + 3]);
            }
    __syncthreads();
#pragma unroll
    for (int o = 0; o < WK; ++o)
        if (grp == o)
#pragma unroll
            for (int f = o * SHARE; f < (o + 1) * SHARE; ++f) {
                v16f &to = acc[f / (NT * 4)][f / 4 % NT];
                float4 v[WK];
#pragma unroll
                for (int n = 0; n < WK; ++n) v[n] = n == o ? make_float4(to[f % 4 * 4], to[f % 4 * 4 + 1], to[f % 4 * 4 + 2], to[f % 4 * 4 + 3]) : *at(o, n, f);
                auto sum = [&](auto get) { return WK == 2 ? get(v[0]) + get(v[1]) : (get(v[0]) + get(v[2 % WK])) + (get(v[1]) + get(v[3 % WK])); };
                to[f % 4 * 4] = sum([](float4 a) { return a.x; });
                to[f % 4 * 4 + 1] = sum([](float4 a) { return a.y; });
                to[f % 4 * 4 + 2] = sum([](float4 a) { return a.z; });
                to[f % 4 * 4 + 3] = sum([](float4 a) { return a.w; });
            }
    __syncthreads();
    // ---- the tile in the output's type through LDS, so that whole rows of it are stored.  Register 4 e + i
    // of lane (r, kg): token r, row 8 e + 4 kg + i of the 32
    constexpr int RW = 32 * MB * WR;                           // rows of the workgroup
    const int size = out_dtype == RB_F32 ? 4 : 2, pitch = RW * size + 16;
#pragma unroll
    for (int o = 0; o < WK; ++o)
        if (grp == o)
#pragma unroll
            for (int f = o * SHARE; f < (o + 1) * SHARE; ++f) {
                const int b = f / (NT * 4), n = f / 4 % NT, e = f % 4;
                const float4 base = *reinterpret_cast<const float4 *>(&row_scale[64 * wr + 32 * b + 8 * e + 4 * kg]);
                uint8_t *const dst = lds + (32 * n + r) * pitch + (32 * (MB * wr + b) + 8 * e + 4 * kg) * size;
                const float v[4] = {acc[b][n][4 * e] * base.x, acc[b][n][4 * e + 1] * base.y, acc[b][n][4 * e + 2] * base.z, acc[b][n][4 * e + 3] * base.w};
                if (out_dtype == RB_F32) {
                    *reinterpret_cast<float4 *>(dst) = make_float4(v[0], v[1], v[2], v[3]);
                } else {
                    uint32_t to[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) to[i] = out_dtype == RB_F16 ? __half_as_ushort(__float2half_rn(v[i])) : f32_to_bf16_rne(v[i]);
                    *reinterpret_cast<uint2 *>(dst) = make_uint2(to[0] | (to[1] << 16), to[2] | (to[3] << 16));
                }
            }
    __syncthreads();
    const int first = id / TB * RW, rows = min(RW, out - first), tokens = min(TOK, T - t0), per16 = 16 / size;
    uint8_t *const Yt = Y + ((size_t)t0 * out + first) * size;
    // 16 bytes at a time whether rows of Y start at multiples of 16 bytes or not (10999 x 4128 at 2048 tokens: element by element 10 % of
    // the call), the end of a row that is no whole piece element by element
    constexpr int PIECES = RW / 8;                             // of two-byte elements; a power of two, as is the number of four-byte ones
    const int chunks = PIECES * 8 / per16;
    for (int i = tid; i < tokens * chunks; i += WAVES * 64) {
        const int t = i / chunks, c = i % chunks;
        uint8_t *const to = Yt + ((size_t)t * out + c * per16) * size;
        const uint8_t *const from = lds + t * pitch + c * 16;
        if ((c + 1) * per16 <= rows) {
            const uint4 v = *reinterpret_cast<const uint4 *>(from);
            __builtin_memcpy(to, &v, 16);
        } else {
            for (int e = 0; e < per16 && c * per16 + e < rows; ++e) {
                if (size == 4) *reinterpret_cast<float *>(to + e * 4) = *reinterpret_cast<const float *>(from + e * 4);
                else *reinterpret_cast<uint16_t *>(to + e * 2) = *reinterpret_cast<const uint16_t *>(from + e * 2);
            }
        }
    }
}

// scales that start at an odd multiple of two bytes, to where 16-byte loads can have them
__global__ __launch_bounds__(256) void align_kernel(const uint16_t *__restrict__ h, uint16_t *__restrict__ to, int n)
{
    for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) to[i] = h[i];
}

// ------------------------------------------------------------------ host ---
// The shapes of a workgroup, and what a round of the device takes with each, in microseconds: `fixed` (launch,
// scales, first loads, sums, stores) and `step` per step of 128 columns per group, for two and for three paths.
// Measured on layers of 256 to 11008 columns (4096 x 11008, 22 or 43 steps, against 4096 x 4096, 8 or 16) with an earlier form of the
// kernel, which now takes 0.7 to 1.25 of the estimate; but all five shapes became faster alike: timed on 50 random layers (256 to 28672 rows, 256 to
// 8128 columns, 71 to 1894 tokens, two and three paths, both types) the one that is picked was the fastest on every one.  A
// round costs the same whether it fills the device or not (11008 x 4096 at 333 tokens, two paths: 172 workgroups of
// 256 x 96 47 us, 129 of 256 x 128 55, 258 of 256 x 64 76, 516 of 128 x 64 75), so the shape with the least sum is taken.
struct Shape { int NT, WR; float fixed, step[2]; };
constexpr Shape SHAPES[] = {{1, 2, 8.f, {1.8f, 2.5f}}, {2, 2, 10.5f, {2.3f, 2.95f}}, {2, 4, 10.f, {1.95f, 2.55f}},
                            {3, 4, 11.5f, {2.25f, 2.9f}}, {4, 4, 13.f, {2.85f, 3.4f}}};
constexpr int N_SHAPES = sizeof(SHAPES) / sizeof(SHAPES[0]);

static int tiles_of(const Shape &s, int out, int T)
{
    return (row_tiles(out) + 4 * s.WR - 1) / (4 * s.WR) * ((T + 32 * s.NT - 1) / (32 * s.NT));
}
static int best_shape(const rb_layer *L, int T, float &least)
{
    const int cus = std::max(1, mx::device_groups()), n128 = (L->in + STEP_COLS - 1) / STEP_COLS;
    int best = 0;
    for (int i = 0; i < N_SHAPES; ++i) {
        const int groups = WAVES / SHAPES[i].WR, rounds = (tiles_of(SHAPES[i], L->out, T) + cus - 1) / cus;
        const float c = (float)rounds * (SHAPES[i].fixed + SHAPES[i].step[L->K - 2] * (float)((n128 + groups - 1) / groups));
        if (i == 0 || c < least) { best = i; least = c; }
    }
    return best;
}

float cost(const rb_layer *L, int T)
{
    float least = 0.f;
    best_shape(L, T, least);
    return least;
}

template <int K, int NT, int WR, bool BF16> static int launch_form(const Args &a, hipStream_t stream)
{
    constexpr int lds = lds_bytes<K, NT, WR>();
    static std::atomic<bool> allowed[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return RB_ERR_HIP;
    if (!allowed[dev].load()) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(gemm_kernel<K, NT, WR, BF16>), hipFuncAttributeMaxDynamicSharedMemorySize, lds) != hipSuccess)
            return RB_ERR_HIP;
        allowed[dev].store(true);
    }
    const int tiles = tiles_of(Shape{NT, WR, 0.f, {0.f, 0.f}}, a.out, a.T);
    hipLaunchKernelGGL((gemm_kernel<K, NT, WR, BF16>), dim3((unsigned)((tiles + 7) / 8 * 8)), dim3(WAVES * 64), lds, stream,
                       address_of(a.bits), address_of(a.h), address_of(a.X), address_of(a.g), address_of(a.Y), a.out, a.in, a.T, a.out_dtype);
    return RB_OK;
}

template <int K, bool BF16> static int launch_shape(const Args &a, int shape, hipStream_t stream)
{
    switch (shape) {
    case 0: return launch_form<K, 1, 2, BF16>(a, stream);
    case 1: return launch_form<K, 2, 2, BF16>(a, stream);
    case 2: return launch_form<K, 2, 4, BF16>(a, stream);
    case 3: return launch_form<K, 3, 4, BF16>(a, stream);
    default: return launch_form<K, 4, 4, BF16>(a, stream);
    }
}

// What a caller is asked for (rb_workspace_bytes): room for the input and, when 256 x 256 tiles
// do not fill whole rounds of the device, for partial sums of the tiles of the last round.  This kernel uses
// the room for the input when the output overlaps it, and the room for the scales when they are not aligned to
// 16 bytes; the size asked for, and with it what rb_linear_gemm_noalloc turns down, is what it was with the
// kernel before this one.
constexpr int BLK = 256;
constexpr size_t SCALES_BYTES = 256, HBLOCK_BYTES = 256;
size_t workspace_bytes(const rb_layer *L, int T)
{
    const int T_pad = (T + BLK - 1) / BLK * BLK, CT = col_tiles(L->in), TB = T_pad / BLK;
    const int tiles = (row_tiles(L->out) + BLK / TILE_ROWS - 1) / (BLK / TILE_ROWS) * TB;
    const int cus = mx::device_groups(), G = cus > 0 ? cus : 256;       // no device (size queries on a host): an MI355X
    const int full = tiles / G * G / TB * TB, tail = tiles - full;
    const int cut = tail > 0 ? std::min(std::min(G / tail, 4), CT) : 1;
    const size_t input = ((size_t)T_pad * CT * TILE_COLS * 2 + 255) / 256 * 256;
    const size_t partial = cut > 1 ? (size_t)cut * T * (L->out - full / TB * BLK) * sizeof(float) : 0;
    return SCALES_BYTES + (size_t)CT * 8 * HBLOCK_BYTES + input + partial;
}

bool supported(const rb_layer *L, int T)
{
    return (L->K == 2 || L->K == 3) && T >= 1 && L->in < MAX_IN;
}

int launch(const rb_layer *L, const void *X, void *Y, int T, int act_dtype, int out_dtype, void *workspace,
           hipStream_t stream)
{
    uint8_t *const room_h = static_cast<uint8_t *>(workspace) + SCALES_BYTES, *const room_x = room_h + (size_t)col_tiles(L->in) * 8 * HBLOCK_BYTES;
    if (overlap(X, input_bytes(L, T), Y, output_bytes(L, T, out_dtype))) {
        copy_aside(X, room_x, input_bytes(L, T), stream);
        X = room_x;
    }
    // (a launch, some 3 us; with eight 2-byte loads in place of one in the kernel 4096 x 4096 at 100 tokens took 43 us
    // where aligned scales take 22, and 28672 x 8192 at 2048 tokens a third longer)
    const uint16_t *h = L->h;
    if ((uintptr_t)h & 15) {
        static_assert(8 * HBLOCK_BYTES >= RB_MAX_K * TILE_COLS * sizeof(uint16_t), "the scales fit");
        const int n = L->K * L->in;
        hipLaunchKernelGGL(align_kernel, dim3((unsigned)std::min(256, (n + 255) / 256)), dim3(256), 0, stream, h, reinterpret_cast<uint16_t *>(room_h), n);
        h = reinterpret_cast<const uint16_t *>(room_h);
    }
    Args a;
    a.bits = static_cast<const uint32_t *>(L->bits);
    a.g = reinterpret_cast<const __half *>(L->g);
    a.h = reinterpret_cast<const __half *>(h);
    a.X = X; a.Y = Y;
    a.out = L->out; a.in = L->in; a.T = T; a.out_dtype = out_dtype;
    float cost;
    const int s = best_shape(L, T, cost);
    const int rc = L->K == 2 ? (act_dtype == RB_BF16 ? launch_shape<2, true>(a, s, stream) : launch_shape<2, false>(a, s, stream))
                             : (act_dtype == RB_BF16 ? launch_shape<3, true>(a, s, stream) : launch_shape<3, false>(a, s, stream));
    if (rc != RB_OK) return rc;
    return hipGetLastError() == hipSuccess ? RB_OK : RB_ERR_HIP;
}

}  // namespace gemm
}  // namespace rb
