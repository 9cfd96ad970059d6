// Few-token kernel of the residual-binary layer: single calls and stacks of a handful to a few dozen
// tokens, two or three paths.  Every op streams its packed weights ONCE for all tokens.
//
// Section 4.1: Y[t] = sum_k g_k (.) (B_k (h_k (.) X[t])), here with the input scale on the side of the
// signs: the left operand of v_mfma_f32_16x16x32_f16 is +-h_k[j] (the stored fp16 scale with the sign
// bit of the weight put in), the right operand is the fp16 activation itself.  Both are exact, so are
// their products, and only fp32 sums round; the activation is shared by the paths, nothing about the
// input is prepared, and an op is one launch.  bfloat16 activations keep their whole range: they go into
// v_mfma_f32_16x16x32_bf16 as they are, against two left operands, as an fp16 scale is the exact sum of two bf16
// values (five vector instructions per four weights and path in place of three and twice the matrix instructions).  Up to 16 tokens only
// where it must be: 128 columns whose values fp16 holds exactly (zeros, 2^-17 up to 65536, which is nearly all there is) are
// multiplied as fp16, the others after them (28672 x 8192 at 5 tokens of bfloat16 27 to 28 us, of fp16 24 to 26; in an earlier
// form of this kernel 34, 47 with two operands throughout, 33 with unchecked fp16 copies).  What bounds it:
//   * a launch of a 4096-wide op moves 4 MB of signs, half a microsecond of HBM time, so it is a
//     chain of latencies (launch, one trip to memory, the matrix instructions, the sum over the
//     wavefronts): the compute units are filled and every wavefront asks for all it needs at once, the
//     output scales of the end included;
//   * the address unit, if activations are fetched in operand order (32 lines a load instruction: 11008
//     columns for one row tile took 14.6 us where the transposition through LDS below took 11, 9.1 now);
//   * beyond that, vector instructions: three per four weights and path (a 64-bit shift for two words and a three-input logic
//     operation for two weights).  A matrix instruction of 512 weights takes 6.7 ns of a SIMD, with the six of its left operand 14.5, of which
//     16 to 17 are reached here; with a shift for each word 16.9 (28672 x 8192 at 16 tokens 27.6 us then and 25.8 so on one card; so 26 to 28 from
//     card to card).
//   * the number of load instructions: one that fetches nothing (past the end, or a second unit asked for ahead of
//     time) takes its turn in the address unit all the same, and asking two units ahead made every launch slower (7B chain
//     at 16 tokens 1.47 ms).
// Shape: a workgroup owns P row tiles (16 rows) and all columns; its wavefronts share out the columns in runs of
// 128 (so that 17 column tiles do not take twice as long as 16), each takes all P row tiles of its columns, so an activation is
// read from memory by one wavefront of the workgroup.  The partial outputs of the wavefronts meet in LDS and are added in
// a fixed order.  Nothing is exchanged between workgroups: no counters, no scratch memory, results do
// not depend on scheduling.  The ops of a stack that do not depend on each other (q/k/v, gate/up of
// a transformer block) run in one launch; dependent ones are ordered by the stream.
//
// Measured (in brackets the form before this one: whole column tiles per wavefront, loads in branches, which made the
// waits coarse and took up to 60 registers more, one workgroup per compute unit): 7B-shaped dependent chain, 128 launches, 1.26 to 1.28 ms
// at 16 tokens (1.37); 13B-shaped, three paths, 32 launches, 6 tokens 0.49 to 0.52 ms (0.62).  Of a launch 1.4 us pass
// between the last wavefront of one and the first of the next, and 1.2 until the first activations are there.  Single calls
// in a graph: 28672 x 8192 at 16 tokens 26 to 28 us (33.5), 10999 x 4128 at 4 7.2 to 7.9 (9.9), 4096 x 4096 at 4 4.5 to 4.8 (5.5), 11008 x 4096 at 48
// 16.3 to 16.9 (28.9), three paths 13824 x 5120 at 48 33.6 to 35.3 (53.8).
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>

#include <algorithm>
#include <atomic>
#include <climits>
#include <cmath>
#include <map>
#include <memory>
#include <mutex>
#include <type_traits>
#include <vector>

#include "rabit.h"
#include "rb_device.h"
#include "rb_internal.h"
#include "rb_layout.h"

namespace rb {
namespace batch {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef unsigned v2u __attribute__((ext_vector_type(2)));
typedef unsigned v3u __attribute__((ext_vector_type(3)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef __bf16 v8b __attribute__((ext_vector_type(8)));

constexpr int STACK_MAX_T = 16;        // tokens of a stack
constexpr int MAX_STAGE_OPS = 8;       // independent ops that share a launch
constexpr int LDS_BYTES = 160 * 1024;  // of a compute unit

// The forms of a workgroup.  Row tiles: as many as fit without spilling (accumulators take 4 P K G registers, sign words 2 P K, staged
// activations 16 G); with four token groups three for two paths and two for three (with a shift per sign word 11008 x 4096 at 64 tokens 18.9 us,
// 26.5 with two; 13824 x 5120, three paths, 39.0 and 54.5 with one; now 17.5 and 37), but not for bfloat16, whose two left operands would spill
// 64 registers (28672 x 8192: 192 us, 124 with two).  Wavefronts: eight, of which two workgroups share a compute unit where 128
// registers are enough, so that one multiplies while the other waits for memory and more workgroups than compute units
// still run at once (28672 x 8192 at 16 tokens: 448 workgroups of four row tiles 26.4 us, with sixteen wavefronts each, in two
// rounds, 29.9); three paths go up to seven row tiles, so that a launch needs one round more often (28672 x 8192 at 16 tokens 38.6 us with four
// in two rounds, 32.7 with seven in one; gate and up of 13824 x 5120 at 6 26.5, 22.5; for two paths, of which two workgroups of four run at
// once, 25.6 and 26.2); sixteen, where 128 registers are enough for them, in a launch that has no second workgroup for a compute unit, from 5120
// columns on (4096 of bfloat16) for two row tiles and more (time of sixteen over that of eight, 9 tokens: one row tile 4128 columns
// 1.00, 11008 0.87; two and three 2080 1.09, 4128 1.01 to 1.04, 1.00 of bfloat16, 6144 0.99, 8192 0.96, 11008 0.98).
__host__ __device__ constexpr bool p_available(int K, int G, int P, bool bf16)
{
    if (P == 1) return true;
    if (G == 1) return K == 2 ? P <= 4 || P == 6 : P <= 7;
    return P * K <= (G == 2 ? 8 : bf16 ? 4 : 6);
}
__host__ __device__ constexpr bool two_share(int K, int G, int P) { return G == 1 ? P * K <= 8 : G == 2 && P == 1; }
__host__ __device__ constexpr bool sixteen_available(int K, int G, int P) { return (G == 1 && P * K <= 8) || (G == 2 && P == 1); }
// Forms in which two left operands at a time, whose words share their shifts, would spill 16 registers (four token groups, where
// matrix instructions are the larger part): 28672 x 8192 at 64 tokens 82 us, 92 so; three paths 105 and 117
__host__ __device__ constexpr bool shifts_in_pairs(int K, int G, int P) { return G < 4 || P * K < 6; }

// One op of a launch: 14 words, which is what a workgroup can be given in registers at its start
struct alignas(64) Op {
    const uint32_t *bits;     // native sign tiles
    const void *x;            // [T][in]
    const uint16_t *h;        // fp16 [K][in]
    const uint16_t *g;        // fp16 [K][out]
    void *y;                  // [T][out]
    int out, in;
    uint32_t tokens;          // T (every entry point turns down more than 65535), element type of y << 16
    uint32_t cut;             // wavefronts of a workgroup, `rest` << 5, `run` << 9: each takes `run` units, the first `rest` one more
    __host__ __device__ int T() const { return (int)(tokens & 0xffffu); }
    __host__ __device__ int out_dtype() const { return (int)(tokens >> 16); }
    __host__ __device__ int waves() const { return (int)(cut & 31u); }
    __host__ __device__ int rest() const { return (int)(cut >> 5 & 15u); }
    __host__ __device__ int run() const { return (int)(cut >> 9); }
};
// Everything a launch needs is passed by value: no table in memory to fetch before the work starts.  The op of a workgroup is its
// blockIdx.y.  The first comes as single arguments, which the compiler has put into registers (build.py asks for it; 7B-shaped chain at 16
// tokens, 128 launches, 1301 us with all in memory, 1273 so; 10999 x 4128 at 7 8.83 and 8.68).  The others are in memory, 64 bytes each, fetched in
// one trip.
struct Others { Op op[MAX_STAGE_OPS - 1]; };
struct Args { Op first; Others others; Op &op(int i) { return i == 0 ? first : others.op[i - 1]; } };

// ------------------------------------------------------------------- kernel ---
// eight values in memory order as the pairs (e, e + 4), e = 0..3: the order in which one shift of a
// native sign word serves both halves of a register
__device__ __forceinline__ uint4 pair_order(uint4 v)
{
    return make_uint4(__builtin_amdgcn_perm(v.z, v.x, 0x05040100u), __builtin_amdgcn_perm(v.z, v.x, 0x07060302u),
                      __builtin_amdgcn_perm(v.w, v.y, 0x05040100u), __builtin_amdgcn_perm(v.w, v.y, 0x07060302u));
}
// an fp16 scale as two bf16 values: the one below it in magnitude and what is left (at most eight bits of
// eleven, then at most three; or one unit, where the scale itself is a bf16 value).  Their sum is exact,
// both have the scale's sign, and neither is zero unless the scale is: an infinite activation gives
// the infinity that its product with the scale is
__device__ __forceinline__ void split_scale(unsigned short h, uint32_t &high, uint32_t &low)
{
    const float f = __half2float(__ushort_as_half(h));
    const uint32_t u = __float_as_uint(f);
    high = (u << 1) != 0u ? (u - 1u) & 0xffff0000u : u;
    low = __float_as_uint(f - __uint_as_float(high));
}
__device__ __forceinline__ void split_scales(uint4 h, uint4 &high, uint4 &low)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t v = reinterpret_cast<const uint32_t *>(&h)[i];
        uint32_t h0, l0, h1, l1;
        split_scale((unsigned short)(v & 0xffffu), h0, l0);
        split_scale((unsigned short)(v >> 16), h1, l1);
        reinterpret_cast<uint32_t *>(&high)[i] = __builtin_amdgcn_perm(h1, h0, 0x07060302u);
        reinterpret_cast<uint32_t *>(&low)[i] = __builtin_amdgcn_perm(l1, l0, 0x07060302u);
    }
}

// loads that return zero past the end of their buffer (NOWHERE always is), so that what is absent of a row, a unit or a row tile needs
// no branch.  Two kinds of branch are left around loads: a uniform one per four tokens (none of which may be there) and the
// lanes of the scales; the waits merge there
constexpr uint32_t NOWHERE = 0x40000000u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer(const void *p, size_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00020000);
}
// the K words of one lane for half a sign tile (path k, columns 32 (lane / 16) .. of the 128)
template <int K> struct Words { uint32_t w[K]; };
template <int K> __device__ __forceinline__ Words<K> load_words(__amdgpu_buffer_rsrc_t rs, uint32_t lane_offset, int offset)
{
    Words<K> r;
    if constexpr (K == 2) {
        const v2u v = __builtin_bit_cast(v2u, __builtin_amdgcn_raw_buffer_load_b64(rs, (int)lane_offset, offset, 0));
        r.w[0] = v.x; r.w[1] = v.y;
    } else {
        const v3u v = __builtin_bit_cast(v3u, __builtin_amdgcn_raw_buffer_load_b96(rs, (int)lane_offset, offset, 0));
        r.w[0] = v.x; r.w[1] = v.y; r.w[2] = v.z;
    }
    return r;
}

// the words of P row tiles two by two, the first of two in the lower half; the last of an odd number with itself, four bits further on
template <int N> struct Pairs { unsigned long long pair[(N + 1) / 2]; };
template <int K, int P> __device__ __forceinline__ Pairs<P * K> pairs_of(const Words<K> (&ws)[P])
{
    Pairs<P * K> r;
#pragma unroll
    for (int n = 0; n < P * K; n += 2) {
        uint32_t lower, upper;
        // copies at this place: ones that the compiler puts at the end of the loop would wait for the next words
        asm volatile("v_mov_b32 %0, %1" : "=&v"(lower) : "v"(ws[n / K].w[n % K]));
        if (n + 1 < P * K) asm volatile("v_mov_b32 %0, %1" : "=&v"(upper) : "v"(ws[(n + 1) / K].w[(n + 1) % K]));
        else upper = lower >> 4;
        r.pair[n / 2] = (unsigned long long)upper << 32 | lower;
    }
    return r;
}
// bfloat16 values whose fp16 values are the same, in pair order; the others are marked in `range`: below 2^-17 in magnitude
// (but zero) or at 65536 and beyond, infinities and NaN
typedef unsigned short v2us __attribute__((ext_vector_type(2)));
struct Bf16Range {
    v2us least = {0xffff, 0xffff}, most = {0, 0};              // of the magnitudes less one (a zero: the largest) and of the magnitudes
    __device__ __forceinline__ void look_at(uint4 v)
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const v2us m = __builtin_bit_cast(v2us, reinterpret_cast<const uint32_t *>(&v)[i] & 0x7fff7fffu);
            least = __builtin_elementwise_min(least, (v2us)(m - (v2us){1, 1}));
            most = __builtin_elementwise_max(most, m);
        }
    }
    __device__ __forceinline__ bool beyond_fp16() const
    {
        return least.x < 0x36ff || least.y < 0x36ff || most.x >= 0x4780 || most.y >= 0x4780;
    }
};
__device__ __forceinline__ uint4 pair_order_as_fp16(uint4 v)
{
    auto pair = [](uint32_t a, uint32_t b) { return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(__uint_as_float(a), __uint_as_float(b))); };
    return make_uint4(pair(v.x << 16, v.z << 16), pair(v.x & 0xffff0000u, v.z & 0xffff0000u),
                      pair(v.y << 16, v.w << 16), pair(v.y & 0xffff0000u, v.w & 0xffff0000u));
}

constexpr int ROW_BYTES = UNIT_COLS * 2;             // a token's fp16 values of the columns that a wavefront stages at a time
__host__ __device__ constexpr int slab_bytes(int K, int G, bool bf16) { return (16 * G + K * (bf16 ? 2 : 1)) * ROW_BYTES; }
// of a wavefront: its slab, then its part of the sums
__host__ __device__ constexpr int wave_bytes(int K, int G, int P, bool bf16) { return slab_bytes(K, G, bf16) > P * G * 1024 ? slab_bytes(K, G, bf16) : P * G * 1024; }

// K paths, G groups of 16 tokens, P row tiles per workgroup of W wavefronts at most, BF16: the activations are bfloat16, WIDE: offsets into
// the input or into the signs of a row tile may reach NOWHERE (1 GiB): 64-bit addresses, loads in branches, one row tile per workgroup
template <int K, int G, int P, int W, bool BF16, bool WIDE>
__global__ __launch_bounds__(W * 64, two_share(K, G, P) && !WIDE ? 4 : 2) void batch_kernel(Address bits, Address x, Address h, Address g, Address y,
                                                                                        int out, int in, uint32_t tokens, uint32_t cut, const Others others)
{
    // bfloat16: fp16 copies of the units that fp16 holds, the others after them as they are.  Beyond one token group looking at a
    // unit costs what the copies save (4096 x 4096 at 24 tokens: 9.3 us with copies unlooked at, 11.5 with the look, 9.2
    // without copies; at 64, 14.2 without copies)
    constexpr bool EITHER = BF16 && G == 1;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];    // a slab per wavefront; then [wavefront][row tile][token][row] sums
    __shared__ __attribute__((aligned(16))) float g_lds[P * K * TILE_ROWS];      // [path][row tile][row]
    Op op = {global_at<const uint32_t>(bits), global_at<const uint8_t>(x), global_at<const uint16_t>(h), global_at<const uint16_t>(g), global_at<uint8_t>(y), out, in, tokens, cut};
    if (blockIdx.y != 0) {
        op = others.op[blockIdx.y - 1];
        // (all of it at once: left to itself the compiler fetches it in four trips, each where it is used first)
        asm volatile("" :: "s"(op.bits), "s"(op.g), "s"(op.h), "s"(op.x), "s"(op.y), "s"(op.out), "s"(op.in), "s"(op.tokens), "s"(op.cut));
    }
    out = op.out;
    in = op.in;
    const int tid = threadIdx.x, lane = tid & 63, nw = op.waves(), threads = nw * 64;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, q = lane >> 4;
    // (calls of more than 64 tokens: blockIdx.z takes 64 of them)
    const int t0 = G == 4 ? (int)blockIdx.z * 64 : 0;
    const int T = G == 4 ? min(op.T() - t0, 64) : op.T();
    const int RT = row_tiles(out), CT = col_tiles(in), rt0 = (int)blockIdx.x * P;
    if (rt0 >= RT) return;                                     // (an op with fewer row tiles than another one of the launch)

    const UnitRun units = unit_run(wave, op.run(), op.rest());
    const int u0 = units.begin, u1 = units.end;
    // ---- staging.  A load instruction fetches 256 contiguous bytes of four tokens (a token per 16 lanes: 16
    // chunks of eight columns), so it touches eight lines; fetched in operand order it would touch 32 and
    // the address unit would bound the kernel.  Chunk 4 q + s (columns 32 q + 8 s ..) of a row goes to position
    // (4 s + q) ^ (row % 16) of the wavefront's own slab: neither these writes nor the operand reads collide
    const int ch = lane & 15, row4 = lane >> 4, pos = (ch & 3) * 4 + (ch >> 2);
    uint8_t *const slab = lds + (size_t)wave * slab_bytes(K, G, BF16);
    const __amdgpu_buffer_rsrc_t x_rs = buffer(static_cast<const uint8_t *>(op.x) + (size_t)t0 * in * 2, (size_t)T * in * 2);
    const __amdgpu_buffer_rsrc_t w_rs = buffer(op.bits + (size_t)rt0 * CT * tile_words(K), (size_t)min(P, RT - rt0) * CT * tile_words(K) * 4);
    uint32_t x_off[4 * G];                                     // (rows of no token are not fetched)
#pragma unroll
    for (int i = 0; i < 4 * G; ++i) x_off[i] = 4 * i + row4 < T ? ((uint32_t)(4 * i + row4) * (uint32_t)in + 8u * (uint32_t)ch) * 2u : NOWHERE;
    const uint16_t *const x_wide = static_cast<const uint16_t *>(op.x) + (size_t)t0 * in;
    const uint32_t h_row = (uint32_t)row4 * (uint32_t)in;
    uint4 xs[4 * G], hs;
    Words<K> ws[P];
    auto real = [&](int u) { return chunk_exists(u, ch, in); };
    // (of a unit that exists: the loads of the scales know no end)
    auto request = [&](int u) {
        const bool some = real(u);
#pragma unroll
        for (int i = 0; i < 4 * G; ++i) {
            if constexpr (WIDE) {
                xs[i] = make_uint4(0u, 0u, 0u, 0u);
                if (4 * i + row4 < T && some) xs[i] = *reinterpret_cast<const uint4 *>(x_wide + (size_t)(4 * i + row4) * in + (size_t)u * UNIT_COLS + 8 * ch);
            } else if (4 * i < T) {
                xs[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(x_rs, (int)(some ? x_off[i] : NOWHERE), u * ROW_BYTES, 0));
            }
        }
        // (the scales need only be 2-byte aligned)
        if (row4 < K) __builtin_memcpy(&hs, op.h + u * UNIT_COLS + (h_row + chunk_scales_at(u, ch, in)), 16);
    };
    const int p_last = min(P, RT - rt0) - 1;
    auto request_words = [&](int u) {
#pragma unroll
        for (int p = 0; p < P; ++p)                            // a row tile past the end of the matrix reads as zero (not stored)
            if constexpr (WIDE) {
                const uint32_t *const w = op.bits + ((size_t)(rt0 + min(p, p_last)) * CT + (u >> 1)) * tile_words(K) + lane * 2 * K + (u & 1) * K;
#pragma unroll
                for (int k = 0; k < K; ++k) ws[p].w[k] = w[k];
            } else {
                ws[p] = load_words<K>(w_rs, (p <= p_last ? 0u : NOWHERE) + (uint32_t)lane * 8u * K, ((min(p, p_last) * CT + (u >> 1)) * tile_words(K) + (u & 1) * K) * 4);
            }
    };
    auto put_x = [&](auto order) {
#pragma unroll
        for (int i = 0; i < 4 * G; ++i)
            if (4 * i < T) *reinterpret_cast<uint4 *>(slab + (4 * i + row4) * ROW_BYTES + ((pos ^ ((4 * i + row4) & 15)) * 16)) = order(xs[i]);
    };
    auto put_h = [&](int m, uint4 v) { *reinterpret_cast<uint4 *>(slab + (16 * G + m * K + row4) * ROW_BYTES + pos * 16) = pair_order(v); };
    auto scales = [&](int u) {
        const uint32_t all = real(u) ? ~0u : 0u;
        return make_uint4(hs.x & all, hs.y & all, hs.z & all, hs.w & all);
    };
    // fp16 activations, or fp16 copies of bfloat16 ones
    auto put = [&](int u) {
        if constexpr (EITHER) put_x([](uint4 v) { return pair_order_as_fp16(v); });
        else put_x([](uint4 v) { return pair_order(v); });
        if (row4 < K) put_h(0, scales(u));
        __builtin_amdgcn_wave_barrier();
    };
    auto put_wide = [&](int u) {
        put_x([](uint4 v) { return pair_order(v); });
        if (row4 < K) {
            uint4 high, low;
            split_scales(scales(u), high, low);
            put_h(0, high);
            put_h(1, low);
        }
        __builtin_amdgcn_wave_barrier();
    };
    auto beyond_fp16 = [&]() {
        Bf16Range range;
#pragma unroll
        for (int i = 0; i < 4 * G; ++i)
            if (4 * i < T) range.look_at(xs[i]);
        return (bool)__any(range.beyond_fp16());
    };
    const int u_first = first_request(units, in);
    request(u_first);
    request_words(u_first);
    // output scales, asked for now, shared through LDS when the sums are there
    constexpr int GV = (P * K * TILE_ROWS + 63) / 64;            // (a workgroup may have one wavefront only)
    uint16_t gval[GV];
#pragma unroll
    for (int i = 0; i < GV; ++i) {
        const int at = tid + i * threads, row = min(rt0 * TILE_ROWS + at % (P * TILE_ROWS), out - 1), k = min(at / (P * TILE_ROWS), K - 1);
        gval[i] = op.g[(size_t)k * out + row];
    }
    v4f acc[P][K][G];
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int g = 0; g < G; ++g) acc[p][k][g] = (v4f){0.f, 0.f, 0.f, 0.f};

    const int x_addr = r * ROW_BYTES + ((q ^ r) * 16), h_addr = 16 * G * ROW_BYTES + q * 16;
    // a unit: TERMS left operands per path and row tile.  Pair (e, e + 4) of the lane's eight columns 8 s .. are the native bits 4 e + s and 16
    // more: shifted to the tops of the two halves, they go into the pair of scales.  One 64-bit shift does it for two words, or
    // for two pairs of one word where the number of words is odd.
    auto contract = [&](auto terms, const Pairs<P * K> &w) {
        constexpr int TERMS = decltype(terms)::value, UNROLL = EITHER && TERMS == 2 ? 1 : 4;
#pragma unroll UNROLL
        for (int s = 0; s < 4; ++s) {
            uint4 hv[K][TERMS];
            v4u b[G];
#pragma unroll
            for (int k = 0; k < K; ++k)
#pragma unroll
                for (int m = 0; m < TERMS; ++m) hv[k][m] = *reinterpret_cast<const uint4 *>(slab + h_addr + (m * K + k) * ROW_BYTES + s * 64);
#pragma unroll
            for (int g = 0; g < G; ++g) b[g] = *reinterpret_cast<const v4u *>(slab + (x_addr ^ (s * 64)) + g * 16 * ROW_BYTES);
            auto multiply = [&](int p, int k, const uint32_t (&at_top)[4]) {
#pragma unroll
                for (int m = 0; m < TERMS; ++m) {
                    v4u a;
#pragma unroll
                    for (int e = 0; e < 4; ++e) a[e] = reinterpret_cast<const uint32_t *>(&hv[k][m])[e] ^ (at_top[e] & 0x80008000u);
#pragma unroll
                    for (int g = 0; g < G; ++g)
                        if constexpr (TERMS == 2) acc[p][k][g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8b, a), __builtin_bit_cast(v8b, b[g]), acc[p][k][g], 0, 0, 0);
                        else acc[p][k][g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(v8h, a), __builtin_bit_cast(v8h, b[g]), acc[p][k][g], 0, 0, 0);
                }
            };
#pragma unroll
            for (int n = 0; n < P * K; n += 2) {
                uint32_t first[4], second[4];
                if constexpr (shifts_in_pairs(K, G, P)) {
                    if (n + 1 < P * K) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) shift_left(w.pair[n / 2], 15 - 4 * e - s, first[e], second[e]);
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; e += 2) shift_left(w.pair[n / 2], 15 - 4 * e - s, first[e], first[e + 1]);
                    }
                    multiply(n / K, n % K, first);
                    if (n + 1 < P * K) multiply((n + 1) / K, (n + 1) % K, second);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) first[e] = (uint32_t)w.pair[n / 2] << (15 - 4 * e - s);
                    multiply(n / K, n % K, first);
#pragma unroll
                    for (int e = 0; e < 4; ++e) second[e] = (uint32_t)(w.pair[n / 2] >> 32) << (15 - 4 * e - s);
                    if (n + 1 < P * K) multiply((n + 1) / K, (n + 1) % K, second);
                }
            }
            if (P * K > 4) __builtin_amdgcn_sched_barrier(0);            // operands of one contraction at a time (registers)
        }
    };
    unsigned long long left = 0;                               // EITHER: the units put off, the last bit for all from number 63 on
#pragma unroll 1
    for (int u = u0; u < u1; ++u) {
        const bool late = EITHER && beyond_fp16();
        if (late) left |= 1ull << min(u - u0, 63);
        else if (BF16 && !EITHER) put_wide(u);
        else put(u);
        const Pairs<P * K> w = pairs_of(ws);
        if (u + 1 < u1) {
            request(u + 1);
            request_words(u + 1);
        }
        if (!late) contract(std::integral_constant<int, BF16 && !EITHER ? 2 : 1>(), w);
        __builtin_amdgcn_wave_barrier();
    }
    if (EITHER && left != 0)                                   // (a bit too many costs a second look)
#pragma unroll 1
        for (int u = u0; u < u1; ++u) {
            if (!(left >> min(u - u0, 63) & 1)) continue;
            request(u);
            if (!beyond_fp16()) continue;
            request_words(u);
            put_wide(u);
            contract(std::integral_constant<int, 2>(), pairs_of(ws));
            __builtin_amdgcn_wave_barrier();
        }
#pragma unroll
    for (int i = 0; i < GV; ++i) {
        const int at = tid + i * threads;
        if (at < P * K * TILE_ROWS) g_lds[at] = __half2float(__ushort_as_half(gval[i]));
    }
    __syncthreads();                                           // the slabs have been read, too: the sums take their place
    float *const part = reinterpret_cast<float *>(lds);

    // ---- partial outputs of this wavefront: path sum with the output scales (Section 4.1).  Lane
    // (r, q) holds token r, rows 4 q .. 4 q + 3 of the row tile.
#pragma unroll
    for (int p = 0; p < P; ++p) {
        v4f gq[K];
#pragma unroll
        for (int k = 0; k < K; ++k) gq[k] = *reinterpret_cast<const v4f *>(&g_lds[(k * P + p) * TILE_ROWS + 4 * q]);
#pragma unroll
        for (int g = 0; g < G; ++g) {
            v4f v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int k = 0; k < K; ++k)
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = __builtin_fmaf(gq[k][i], acc[p][k][g][i], v[i]);
            *reinterpret_cast<v4f *>(part + ((wave * P + p) * G + g) * 256 + r * 16 + 4 * q) = v;
        }
    }
    __syncthreads();
    // ---- add the wavefronts in order, round, store
    for (int idx = tid; idx < P * G * 256; idx += threads) {
        const int p = idx / (G * 256), t = idx / 16 % (G * 16), row = (rt0 + p) * TILE_ROWS + idx % 16;
        float s = 0.f;
        for (int v = 0; v < nw; ++v) s += part[v * (P * G * 256) + idx];
        if (t < T && row < out) store_out(op.y, op.out_dtype(), (size_t)(t0 + t) * out + row, s);
    }
}

// ------------------------------------------------------------------ host ---
constexpr int ROW_TILES_PER_WG[] = {1, 2, 3, 4, 5, 6, 7};

// Row tiles per workgroup and its wavefronts.  Beyond NARROW_UNITS of 128 columns: eight wavefronts, row tiles by what the busiest compute
// unit takes, `each` workgroups in rounds of the one or two that run at once.  In units of a row tile's work (0.1 us per column tile) a workgroup
// costs 0.6 more (its activations, the sum) and a round 33 / column tiles (3.3 us: the latencies).  (16 tokens, two paths, us for 1, 2, 3, 4, 6
// row tiles: 12288 x 4096 9.7 9.2 7.8 8.6 11.6; 22016 x 4096 17.6 13.2 11.8 14.7 11.8; 28672 x 8192 39.3 30.8 30.1 26.3 37.9.)  The constants are
// those of a form with a shift per sign word; of 48 three-path layers of 1056 to 10528 columns they still pick one within 3 % of the best in 46 (22016 x
// 3616 at 2 tokens 14.5 us, with two row tiles 13.5).  Sixteen wavefronts: see above.
// Narrower layers leave room for several small workgroups on a compute unit, whose latencies then overlap, and what a workgroup pays for
// its sums is shared by fewer wavefronts.  Microseconds of a round of them, for P row tiles and G token groups: 1.5, per unit of a
// wavefront 0.7 + 0.1 P G, for the sums 0.5 P G / wavefronts.  (us by the rule above and by this one, with a shift per sign word: 28672 x 512
// at 33 tokens 16.9 and 10.9, by this one now 10.3; three paths, 28672 x 1024 at 24 21.2 and 16.6, now 11.6, 5000 x 32 at 64 11.3 and 7.2, now 6.7.
// Of the forms measured for 32 to 1024 columns at 9, 24 and 48 tokens it picked one that was 1 % slower than the best in the mean; now, 108
// three-path layers at 1 to 16 tokens, 3 %, 18 % at most.)
// Five to seven row tiles of three paths are no part of that: each row tile more costs such a workgroup 0.6 to 1.1 us, not the 0.1 to 0.2 per unit
// that the rule counts (2048 x 640 at 5 tokens, one to seven: 3.1 4.0 4.9 5.4 6.2 7.2 8.2; 28672 x 704 at 6 with seven 8.5, with the two chosen
// without them 6.6; of 48 sizes at which it chose them four were 9 to 14 % faster with them, most 5 to 28 % slower).
constexpr int NARROW_UNITS = 8;
struct Form { int P, nw; double cost; };
static Form form_of(const int *RT, int nops, int units, int K, int G, int blocks, bool bf16)
{
    const int cus = std::max(1, mx::device_groups()), CT = (units + 1) / 2;
    auto groups = [&](int P) {
        int n = 0;
        for (int i = 0; i < nops; ++i) n += (RT[i] + P - 1) / P;
        return n * blocks;
    };
    Form best = {0, 0, 0.0};
    for (int P : ROW_TILES_PER_WG) {
        if (!p_available(K, G, P, bf16)) continue;
        const int each = (groups(P) + cus - 1) / cus, at_once = two_share(K, G, P) ? 2 : 1;
        if (units > NARROW_UNITS) {
            const double cost = each * (P + 0.6) + (each + at_once - 1) / at_once * 33.0 / CT;
            if (best.P == 0 || cost < best.cost) best = {P, sixteen_available(K, G, P) && each <= 1 && (P == 1 || units >= (bf16 ? 32 : 40)) ? 16 : 8, cost};
        } else if (P * K <= 12) {
            for (int nw = 1; nw < 2 * units; nw *= 2) {
                const int waves = std::min(nw, units);
                const int resident = std::max(1, std::min(8 * at_once / waves, LDS_BYTES / (waves * wave_bytes(K, G, P, bf16) + P * K * TILE_ROWS * 4)));
                const double cost = (each + resident - 1) / resident * (1.5 + (units + waves - 1) / waves * (0.7 + 0.1 * P * G) + 0.5 * P * G / waves);
                if (best.P == 0 || cost < best.cost) best = {P, waves, cost};
            }
        }
    }
    return best;
}

template <int K, int G, int P, int W, bool BF16, bool WIDE = false>
static int launch_form(const Args &args, int nops, int groups, int nw, hipStream_t stream)
{
    constexpr int per_wave = wave_bytes(K, G, P, BF16), lds_max = W * per_wave;
    if (lds_max + P * K * TILE_ROWS * (int)sizeof(float) > 64 * 1024) {
        static std::atomic<bool> allowed[64];
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return RB_ERR_HIP;
        if (!allowed[dev].load()) {
            if (hipFuncSetAttribute(reinterpret_cast<const void *>(batch_kernel<K, G, P, W, BF16, WIDE>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    lds_max) != hipSuccess)
                return RB_ERR_HIP;
            allowed[dev].store(true);
        }
    }
    hipLaunchKernelGGL((batch_kernel<K, G, P, W, BF16, WIDE>), dim3((unsigned)groups, (unsigned)nops, (unsigned)(G == 4 ? (args.first.T() + 63) / 64 : 1)), dim3((unsigned)(nw * 64)), nw * per_wave, stream,
                       address_of(args.first.bits), address_of(args.first.x), address_of(args.first.h), address_of(args.first.g), address_of(args.first.y), args.first.out, args.first.in, args.first.tokens, args.first.cut, args.others);
    return RB_OK;
}

template <int K, int G, int P, bool BF16>
static int launch_waves(const Args &args, int nops, int groups, int nw, hipStream_t stream)
{
    if constexpr (sixteen_available(K, G, P))
        if (nw > 8) return launch_form<K, G, P, 16, BF16>(args, nops, groups, nw, stream);
    return launch_form<K, G, P, 8, BF16>(args, nops, groups, nw, stream);
}

template <int K, int G, bool BF16>
static int launch_p(const Args &args, int nops, int P, int groups, int nw, bool wide, hipStream_t stream)
{
    if (wide) return launch_form<K, G, 1, G == 1 ? 16 : 8, BF16, true>(args, nops, groups, nw, stream);
    switch (P) {
    case 1: return launch_waves<K, G, 1, BF16>(args, nops, groups, nw, stream);
    case 2: if constexpr (p_available(K, G, 2, BF16)) return launch_waves<K, G, 2, BF16>(args, nops, groups, nw, stream); break;
    case 3: if constexpr (p_available(K, G, 3, BF16)) return launch_waves<K, G, 3, BF16>(args, nops, groups, nw, stream); break;
    case 4: if constexpr (p_available(K, G, 4, BF16)) return launch_waves<K, G, 4, BF16>(args, nops, groups, nw, stream); break;
    case 5: if constexpr (p_available(K, G, 5, BF16)) return launch_waves<K, G, 5, BF16>(args, nops, groups, nw, stream); break;
    case 6: if constexpr (p_available(K, G, 6, BF16)) return launch_waves<K, G, 6, BF16>(args, nops, groups, nw, stream); break;
    default: if constexpr (p_available(K, G, 7, BF16)) return launch_waves<K, G, 7, BF16>(args, nops, groups, nw, stream); break;
    }
    return RB_ERR_UNSUPPORTED;
}

static int token_groups(int T) { return T <= 16 ? 1 : T <= 32 ? 2 : 4; }

// The kernel keeps 32-bit offsets into the input of up to 64 tokens and into the signs of a workgroup's row tiles, both below NOWHERE; where
// they may not fit its WIDE form runs (256 x 2^24 at 3 tokens 7.6 ms, on the generic kernel 40; 64 x 2^24 at 16 13.2 and 39.8)
static bool offsets_fit(int in, int T) { return in < 1 << 24 && (size_t)std::min(T, 64) * in * 2 < NOWHERE; }

// one launch: the first nops ops of `args`, all of K paths and T tokens; P row tiles per workgroup, `groups` workgroups
// for the op with the most row tiles
struct Shape { int K, T, nops, P, groups, nw; bool wide; };
static Shape shape_of(Args &args, int nops, int K, bool bf16)
{
    int RT[MAX_STAGE_OPS], units = 1;
    Shape s = {K, args.first.T(), nops, 0, 0, 0, false};
    for (int i = 0; i < nops; ++i) {
        RT[i] = row_tiles(args.op(i).out);
        units = std::max(units, units_of(args.op(i).in));
        s.wide = s.wide || !offsets_fit(args.op(i).in, s.T);
    }
    const int G = token_groups(s.T);
    const Form form = s.wide ? Form{1, G == 1 ? 16 : 8, 0.0} : form_of(RT, nops, units, K, G, (s.T + 63) / 64, bf16);
    s.P = form.P;
    s.nw = std::min(units, form.nw);
    for (int i = 0; i < nops; ++i) s.groups = std::max(s.groups, (RT[i] + s.P - 1) / s.P);
    for (int i = 0; i < nops; ++i) {
        const int n = units_of(args.op(i).in);
        args.op(i).cut = (uint32_t)(n / s.nw) << 9 | (uint32_t)(n % s.nw) << 5 | (uint32_t)s.nw;
    }
    return s;
}

template <bool BF16> static int launch_shape(const Args &args, const Shape &s, hipStream_t stream)
{
    const int G = token_groups(s.T);
    if (s.K == 2)
        return G == 1 ? launch_p<2, 1, BF16>(args, s.nops, s.P, s.groups, s.nw, s.wide, stream)
             : G == 2 ? launch_p<2, 2, BF16>(args, s.nops, s.P, s.groups, s.nw, s.wide, stream)
                      : launch_p<2, 4, BF16>(args, s.nops, s.P, s.groups, s.nw, s.wide, stream);
    return G == 1 ? launch_p<3, 1, BF16>(args, s.nops, s.P, s.groups, s.nw, s.wide, stream)
         : G == 2 ? launch_p<3, 2, BF16>(args, s.nops, s.P, s.groups, s.nw, s.wide, stream)
                  : launch_p<3, 4, BF16>(args, s.nops, s.P, s.groups, s.nw, s.wide, stream);
}

static Op make_op(const rb_layer &L, const void *x, void *y, int T, int out_dtype)
{
    Op o = {};
    o.bits = static_cast<const uint32_t *>(L.bits);
    o.g = L.g; o.h = L.h;
    o.x = x; o.y = y;
    o.out = L.out; o.in = L.in;
    o.tokens = (uint32_t)T | (uint32_t)out_dtype << 16;
    return o;
}

// (calls and stacks of at most this size are this file's)
static bool sized(const rb_layer *L, int T, int max_T)
{
    return (L->K == 2 || L->K == 3) && T >= 1 && T <= max_T && L->in % 32 == 0 && (size_t)T * L->in < (size_t)1 << 32;
}

bool call_sized(const rb_layer *L, int T) { return sized(L, T, CALL_MAX_T); }

// More than CALL_MAX_T tokens: 64 of them per workgroup, where the workgroups of a call do not outnumber the compute units (in a second
// round the many-token kernel is always the faster one).  Microseconds, launch included: 6.5 and so much per column tile, measured on
// layers of 800 to 11008 columns; or 6.5 and the time in which the workgroups of different rows, on eight dies with caches of their own, fetch
// the activations, 6.2 TB/s (300 rows at 2000 tokens: 2048 columns 16.4 us, 28672 columns 123; the many-token kernel 12.4 and 101).  The
// constants are those of a form with a shift per sign word: estimates are 1.1 to 1.4 times what it takes now (launch_many has the choice that results)
float blocks_cost(const rb_layer *L, int T, int act_dtype)
{
    static constexpr float per_tile[2][2][3] = {{{0.46f, 0.69f, 0.8f}, {0.57f, 0.95f, 0.f}}, {{0.5f, 0.85f, 0.f}, {0.67f, 0.f, 0.f}}};
    const bool bf16 = act_dtype == RB_BF16;
    if (!sized(L, T, INT_MAX) || !offsets_fit(L->in, T)) return INFINITY;
    for (int P = 1; P <= 3 && p_available(L->K, 4, P, bf16); ++P) {
        const int groups = (row_tiles(L->out) + P - 1) / P;
        if ((long long)groups * ((T + 63) / 64) > mx::device_groups()) continue;
        const float fetch = (float)std::min(groups, 8) * (float)input_bytes(L, T) * (1.f / 6.2e6f);
        return 6.5f + std::max(per_tile[L->K - 2][bf16][P - 1] * (float)col_tiles(L->in), fetch);
    }
    return INFINITY;
}

int launch_call(const rb_layer *L, const void *X, void *Y, int T, int act_dtype, int out_dtype, void *workspace,
                size_t workspace_bytes, hipStream_t stream)
{
    // (where nothing is asked for the output must not overlap the input)
    if (single_few_has_room(L, T) && overlap(X, input_bytes(L, T), Y, output_bytes(L, T, out_dtype))) {
        if (!workspace || workspace_bytes < aside_bytes(L, T)) return RB_ERR_WORKSPACE;
        copy_aside(X, workspace, input_bytes(L, T), stream);
        X = workspace;
    }
    Args args = {};
    args.first = make_op(*L, X, Y, T, out_dtype);
    const Shape s = shape_of(args, 1, L->K, act_dtype == RB_BF16);
    const int rc = act_dtype == RB_BF16 ? launch_shape<true>(args, s, stream) : launch_shape<false>(args, s, stream);
    if (rc != RB_OK) return rc;
    return hipGetLastError() == hipSuccess ? RB_OK : RB_ERR_HIP;
}

bool layer_supported(const rb_layer *L, int T) { return sized(L, T, STACK_MAX_T); }

// A plan lives on the host: the kernel needs nothing in device memory besides the buffers.  The
// workspace is the name it is run by, and holds the input of an op whose output overlaps it.
size_t plan_workspace_bytes(const rb_layer *layers, int n_layers, int T)
{
    size_t need = 256;
    for (int l = 0; l < n_layers; ++l) need = std::max(need, aside_bytes(&layers[l], T));
    return need;
}

struct Launch { Args args; Shape shape; const void *aside; size_t aside_bytes; };     // aside: an input to be moved to the workspace first
struct Prepared { std::vector<Launch> launches; size_t need = 256; };
static std::mutex g_mutex;
static std::map<const void *, std::shared_ptr<const Prepared>> g_prepared;

int prepare_plan(const rb_layer *layers, const rb_stack_op *sops, int n_ops, uint16_t *const *bufs, int T,
                 void *workspace, size_t workspace_bytes_)
{
    if (T < 1 || T > STACK_MAX_T) return RB_ERR_UNSUPPORTED;
    auto pr = std::make_shared<Prepared>();
    for (int n = 0; n < n_ops; ++n) pr->need = std::max(pr->need, plan_workspace_bytes(&layers[sops[n].layer], 1, T));
    if (!workspace || workspace_bytes_ < pr->need) return RB_ERR_WORKSPACE;
    // an op that reads another one's output reads all of it
    std::map<int, int> width;
    for (int n = 0; n < n_ops; ++n) {
        const rb_layer &L = layers[sops[n].layer];
        if (!layer_supported(&L, T)) return RB_ERR_UNSUPPORTED;
        const auto it = width.find(sops[n].src);
        if (it != width.end() && it->second != L.in) return RB_ERR_SHAPE;
        width[sops[n].dst] = L.out;
    }
    // launches: runs of consecutive ops of one K that neither read nor overwrite each other.  Memory
    // decides, not the buffers' indices: two of them may overlap.  An op that overwrites its own input gets a launch of
    // its own and reads a copy
    struct Span { const void *at; size_t bytes; };
    auto src = [&](int n) { return Span{bufs[sops[n].src], input_bytes(&layers[sops[n].layer], T)}; };
    auto dst = [&](int n) { return Span{bufs[sops[n].dst], output_bytes(&layers[sops[n].layer], T, RB_F16)}; };
    auto meet = [](Span a, Span b) { return overlap(a.at, a.bytes, b.at, b.bytes); };
    for (int op0 = 0; op0 < n_ops;) {
        Args args = {};
        int nops = 0;
        const int K = layers[sops[op0].layer].K;
        for (int n = op0; n < n_ops && nops < MAX_STAGE_OPS; ++n) {
            const rb_layer &L = layers[sops[n].layer];
            bool conflict = L.K != K || (n > op0 && (meet(src(n), dst(n)) || meet(src(op0), dst(op0))));
            for (int m = op0; m < n; ++m)
                if (meet(dst(m), src(n)) || meet(dst(m), dst(n)) || meet(src(m), dst(n))) conflict = true;
            if (conflict) break;
            args.op(nops++) = make_op(L, bufs[sops[n].src], bufs[sops[n].dst], T, RB_F16);
        }
        const Shape shape = shape_of(args, nops, K, false);
        Launch l = {args, shape, nullptr, 0};
        if (meet(src(op0), dst(op0))) {
            l.aside = src(op0).at;
            l.aside_bytes = src(op0).bytes;
            l.args.first.x = workspace;
        }
        pr->launches.push_back(l);
        op0 += nops;
    }
    std::lock_guard<std::mutex> lock(g_mutex);
    g_prepared[workspace] = std::move(pr);
    return RB_OK;
}

// RB_ERR_UNSUPPORTED: the workspace holds no plan of this kind
int launch_plan(void *workspace, size_t workspace_bytes_, hipStream_t stream)
{
    std::shared_ptr<const Prepared> pr;
    {
        std::lock_guard<std::mutex> lock(g_mutex);
        const auto it = g_prepared.find(workspace);
        if (it == g_prepared.end()) return RB_ERR_UNSUPPORTED;
        pr = it->second;
    }
    if (workspace_bytes_ < pr->need) return RB_ERR_WORKSPACE;
    for (const Launch &l : pr->launches) {
        if (l.aside) copy_aside(l.aside, workspace, l.aside_bytes, stream);
        const int rc = launch_shape<false>(l.args, l.shape, stream);
        if (rc != RB_OK) return rc;
    }
    return hipGetLastError() == hipSuccess ? RB_OK : RB_ERR_HIP;
}

bool has_plan(const void *workspace)
{
    std::lock_guard<std::mutex> lock(g_mutex);
    return g_prepared.find(workspace) != g_prepared.end();
}

void forget_plan(const void *workspace)
{
    std::lock_guard<std::mutex> lock(g_mutex);
    g_prepared.erase(workspace);
}

}  // namespace batch
}  // namespace rb
