// Few-token kernel of the residual-binary layer: single calls and stacks of a handful to a few dozen
// tokens, two or three paths.  Every op streams its packed weights ONCE for all tokens.
//
// Section 4.1: Y[t] = sum_k g_k (.) (B_k (h_k (.) X[t])), here with the input scale on the side of the
// signs: the left operand of v_mfma_f32_16x16x32_f16 is +-h_k[j] (the stored fp16 scale with the sign
// bit of the weight put in), the right operand is the fp16 activation itself.  Both are exact, so are
// their products, and only fp32 sums round; the activation is shared by the paths, nothing about the
// input is prepared, and an op is one launch.  bfloat16 activations keep their whole range: they go into
// v_mfma_f32_16x16x32_bf16 as they are, against two left operands, as an fp16 scale is the exact sum of two bf16
// values (three vector instructions in place of two and twice the matrix instructions).  Up to 16 tokens only
// where it must be: 128 columns whose values fp16 holds exactly (zeros, 2^-17 up to 65536, which is nearly all there is) are
// multiplied as fp16, the others after them (28672 x 8192 at 5 tokens 34 us, 47 with two operands throughout, 33 with
// unchecked fp16 copies).  What bounds it:
//   * a launch of a 4096-wide op moves 4 MB of signs, half a microsecond of HBM time, so it is a
//     chain of latencies (launch, one trip to memory, the matrix instructions, the sum over the
//     wavefronts): the compute units are filled and every wavefront asks for all it needs at once, the
//     output scales of the end included;
//   * the address unit, if activations are fetched in operand order (32 lines a load instruction: 11008
//     columns for one row tile took 14.6 us, the transposition through LDS below takes 11);
//   * beyond that, vector instructions: two per two weights and path (a shift and one three-input logic
//     operation), where the matrix instructions of 16 tokens take a third of their time.
// Shape: a workgroup owns P row tiles (16 rows) and all columns; its up to sixteen wavefronts share out the
// column tiles, each takes all P row tiles of its columns, so an activation is read from memory by
// one wavefront of the workgroup.  The partial outputs of the wavefronts meet in LDS and are added in
// a fixed order.  Nothing is exchanged between workgroups: no counters, no scratch memory, results do
// not depend on scheduling.  The ops of a stack that do not depend on each other (q/k/v, gate/up of
// a transformer block) run in one launch; dependent ones are ordered by the stream.
//
// Measured: 7B-shaped dependent chain, 128 launches, 1.30 ms at 8 tokens and 1.37 ms at 16 (activations in operand
// order, the output scales fetched at the end: 1.42 and 1.61; bf8 term expansions of the activations in LDS, which
// this kernel replaced: 2.51 and 3.09); a launch takes 6.3 us (4096 x 4096, one row tile per workgroup) to 16 us
// (2 x 11008 x 4096, six), of which a dependent launch by itself is 4.7.  Single calls: 4096 x 11008
// with three paths at 16 tokens 12.7 us, 10999 x 4128 with two at 7 tokens 9.7 us, of bfloat16 10.7.
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>

#include <algorithm>
#include <atomic>
#include <climits>
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
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef __bf16 v8b __attribute__((ext_vector_type(8)));

constexpr int STACK_MAX_T = 16;        // tokens of a stack
constexpr int MAX_STAGE_OPS = 8;       // independent ops that share a launch

// Wavefronts of a workgroup at most, and row tiles per workgroup: accumulators take 4 P K G
// registers, sign words 2 P K, staged activations 16 G, of 128 with sixteen wavefronts per compute unit
// and 256 with eight (two paths, six row tiles, 16 tokens: 28.6 us a launch of 2 x 11008 x 4096 with sixteen, which
// spills, 16.2 with eight; four row tiles, 8 tokens, 7B chain: the same either way).  Two paths, four token groups, two row
// tiles spill 14 registers and are worth it: 8192 x 8192 at 64 tokens 30.4 us, 39.0 with one row tile
__host__ __device__ constexpr int max_waves(int K, int G, int P) { return G == 1 && P * K <= 8 ? 16 : 8; }
__host__ __device__ constexpr bool p_available(int K, int G, int P) { return P == 1 || P * K <= (G == 1 ? 12 : G == 2 ? 6 : 4); }

struct Op {
    const uint32_t *bits;     // native sign tiles
    const uint16_t *g;        // fp16 [K][out]
    const uint16_t *h;        // fp16 [K][in]
    const void *x;            // [T][in]
    void *y;                  // [T][out]
    int out, in;
    int h_aligned;            // h starts at a multiple of 16 bytes (its rows then do too)
    int pad_;
};
// everything a launch needs, passed by value: no table in memory to fetch before the work starts.  What
// decides which op a workgroup belongs to comes first, in one piece: it costs one trip to the arguments, the op another
struct Args {
    int T, out_dtype, nops;
    int wg0[MAX_STAGE_OPS];   // first workgroup of each op (past the last op: more than there are)
    int pad_[5];
    Op op[MAX_STAGE_OPS];
};

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

// the 2 K words (word c * K + k: path k, columns 128 c + 32 (lane / 16) ..) of one lane of a sign tile
template <int K> struct Words { uint32_t w[2 * K]; };
template <int K> __device__ __forceinline__ Words<K> load_words(const uint32_t *p)
{
    Words<K> r;
    if constexpr (K == 2) {
        const v4u v = __builtin_nontemporal_load(reinterpret_cast<const v4u *>(p));
        r.w[0] = v.x; r.w[1] = v.y; r.w[2] = v.z; r.w[3] = v.w;
    } else {
#pragma unroll
        for (int i = 0; i < K; ++i) {
            const v2u v = __builtin_nontemporal_load(reinterpret_cast<const v2u *>(p) + i);
            r.w[2 * i] = v.x; r.w[2 * i + 1] = v.y;
        }
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

constexpr int UNIT_COLS = 128, ROW_BYTES = 256;      // columns a wavefront stages at a time; a token's fp16 values of them
template <int K, int G, bool BF16> __host__ __device__ constexpr int slab_bytes() { return (16 * G + K * (BF16 ? 2 : 1)) * ROW_BYTES; }

// K paths, G groups of 16 tokens, P row tiles per workgroup, BF16: the activations are bfloat16
template <int K, int G, int P, bool BF16>
__global__ __launch_bounds__(max_waves(K, G, P) * 64, 1) void batch_kernel(const Args args)
{
    constexpr bool AHEAD = P * K <= (G == 1 ? 6 : 4) && G <= 2;       // registers for the sign words of the next column tile
    // bfloat16: fp16 copies of the units that fp16 holds, the others after them as they are.  Beyond one token group looking at a
    // unit costs what the copies save (4096 x 4096 at 24 tokens: 9.3 us with copies unlooked at, 11.5 with the look, 9.2
    // without copies; at 64, 14.2 without copies)
    constexpr bool EITHER = BF16 && G == 1;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];    // a slab per wavefront; then [wavefront][row tile][token][row] sums
    __shared__ __attribute__((aligned(16))) float g_lds[P * K * TILE_ROWS];      // [path][row tile][row]
    const int tid = threadIdx.x, lane = tid & 63, nw = (int)blockDim.x >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, q = lane >> 4;
    int o = 0, first = 0;
#pragma unroll
    for (int i = 1; i < MAX_STAGE_OPS; ++i)
        if ((int)blockIdx.x >= args.wg0[i]) { o = i; first = args.wg0[i]; }
    const Op &op = args.op[o];
    const int out = op.out, in = op.in, T = args.T;
    const int RT = row_tiles(out), CT = col_tiles(in);
    const int rt0 = ((int)blockIdx.x - first) * P;

    // the row tiles of this workgroup; one past the end of the matrix reads the last one (not stored)
    const uint32_t *bits[P];                                   // (uniform: the lane's offset is added at the load)
#pragma unroll
    for (int p = 0; p < P; ++p) bits[p] = op.bits + (size_t)min(rt0 + p, RT - 1) * CT * tile_words(K);
    const uint32_t lane_words = (uint32_t)lane * 2u * K;

    Words<K> w[P];
    if (wave < CT)
#pragma unroll
        for (int p = 0; p < P; ++p) w[p] = load_words<K>(bits[p] + (size_t)wave * tile_words(K) + lane_words);

    // ---- staging.  A load instruction fetches 256 contiguous bytes of four tokens (a token per 16 lanes: 16
    // chunks of eight columns), so it touches eight lines; fetched in operand order it would touch 32 and
    // the address unit would bound the kernel.  Chunk 4 q + s (columns 32 q + 8 s ..) of a row goes to position
    // (4 s + q) ^ (row % 16) of the wavefront's own slab: neither these writes nor the operand reads collide
    const int ch = lane & 15, row4 = lane >> 4, pos = (ch & 3) * 4 + (ch >> 2);
    uint8_t *const slab = lds + (size_t)wave * slab_bytes<K, G, BF16>();
    uint32_t x_off[4 * G];
#pragma unroll
    for (int i = 0; i < 4 * G; ++i) x_off[i] = (uint32_t)min(4 * i + row4, T - 1) * (uint32_t)in + 8u * (uint32_t)ch;
    uint4 xs[4 * G], hs;
    auto request = [&](int j0) {
        const bool real = j0 + 8 * ch < in;                    // in % 32 == 0: all eight columns or none
        const uint16_t *const x = static_cast<const uint16_t *>(op.x) + j0;
#pragma unroll
        for (int i = 0; i < 4 * G; ++i) {
            xs[i] = make_uint4(0u, 0u, 0u, 0u);
            if (4 * i < T && real) xs[i] = *reinterpret_cast<const uint4 *>(x + x_off[i]);       // (rows of no token are not looked at)
        }
        hs = make_uint4(0u, 0u, 0u, 0u);
        if (row4 < K && real) {
            const uint16_t *const h = op.h + (size_t)row4 * in + j0 + 8 * ch;
            if (op.h_aligned) hs = *reinterpret_cast<const uint4 *>(h);
            else                                               // the scales need only be 2-byte aligned
                hs = make_uint4((uint32_t)h[0] | (uint32_t)h[1] << 16, (uint32_t)h[2] | (uint32_t)h[3] << 16,
                                (uint32_t)h[4] | (uint32_t)h[5] << 16, (uint32_t)h[6] | (uint32_t)h[7] << 16);
        }
    };
    auto put_x = [&](auto order) {
#pragma unroll
        for (int i = 0; i < 4 * G; ++i) {
            const int row = 4 * i + row4;
            if (4 * i < T) *reinterpret_cast<uint4 *>(slab + row * ROW_BYTES + ((pos ^ (row & 15)) * 16)) = order(xs[i]);
        }
    };
    auto put_h = [&](int m, uint4 v) { *reinterpret_cast<uint4 *>(slab + (16 * G + m * K + row4) * ROW_BYTES + pos * 16) = pair_order(v); };
    // fp16 activations, or fp16 copies of bfloat16 ones
    auto put = [&]() {
        if constexpr (EITHER) put_x([](uint4 v) { return pair_order_as_fp16(v); });
        else put_x([](uint4 v) { return pair_order(v); });
        if (row4 < K) put_h(0, hs);
        __builtin_amdgcn_wave_barrier();
    };
    auto put_wide = [&]() {
        put_x([](uint4 v) { return pair_order(v); });
        if (row4 < K) {
            uint4 high, low;
            split_scales(hs, high, low);
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
    if (wave < CT) request(wave * TILE_COLS);
    // output scales, asked for now, shared through LDS when the sums are there
    constexpr int GV = (P * K * TILE_ROWS + 63) / 64;            // (a workgroup may have one wavefront only)
    uint16_t gval[GV];
#pragma unroll
    for (int i = 0; i < GV; ++i) {
        const int at = tid + i * (int)blockDim.x, row = min(rt0 * TILE_ROWS + at % (P * TILE_ROWS), out - 1), k = min(at / (P * TILE_ROWS), K - 1);
        gval[i] = 0;
        if ((int)blockDim.x * i < P * K * TILE_ROWS) gval[i] = op.g[(size_t)k * out + row];
    }
    v4f acc[P][K][G];
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int g = 0; g < G; ++g) acc[p][k][g] = (v4f){0.f, 0.f, 0.f, 0.f};

    const int x_addr = r * ROW_BYTES + ((q ^ r) * 16), h_addr = 16 * G * ROW_BYTES + q * 16;
    // a unit: TERMS left operands per path and row tile
    auto contract = [&](auto terms, int c) {
        constexpr int TERMS = decltype(terms)::value, UNROLL = EITHER && TERMS == 2 ? 1 : 4;
#pragma unroll UNROLL
        for (int s = 0; s < 4; ++s) {
            v4u b[G];
            uint4 hv[K][TERMS];
#pragma unroll
            for (int k = 0; k < K; ++k)
#pragma unroll
                for (int m = 0; m < TERMS; ++m) hv[k][m] = *reinterpret_cast<const uint4 *>(slab + h_addr + (m * K + k) * ROW_BYTES + s * 64);
#pragma unroll
            for (int g = 0; g < G; ++g) b[g] = *reinterpret_cast<const v4u *>(slab + (x_addr ^ (s * 64)) + g * 16 * ROW_BYTES);
#pragma unroll
            for (int k = 0; k < K; ++k)
#pragma unroll
                for (int p = 0; p < P; ++p)
#pragma unroll
                    for (int m = 0; m < TERMS; ++m) {
                        // pair (e, e + 4) of the lane's eight columns 8 s ..: native bits 4 e + s and 16 more
                        v4u a;
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            a[e] = reinterpret_cast<const uint32_t *>(&hv[k][m])[e] ^ ((w[p].w[c * K + k] << (15 - 4 * e - s)) & 0x80008000u);
#pragma unroll
                        for (int g = 0; g < G; ++g)
                            if constexpr (TERMS == 2) acc[p][k][g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8b, a), __builtin_bit_cast(v8b, b[g]), acc[p][k][g], 0, 0, 0);
                            else acc[p][k][g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(v8h, a), __builtin_bit_cast(v8h, b[g]), acc[p][k][g], 0, 0, 0);
                    }
            if (P * K > 4) __builtin_amdgcn_sched_barrier(0);            // operands of one contraction at a time (registers)
        }
    };
    unsigned long long left = 0;                               // EITHER: the units put off, the last bit for all from number 63 on
    for (int ct = wave; ct < CT; ct += nw) {
        Words<K> next[P];
        if (AHEAD && ct + nw < CT)
#pragma unroll
            for (int p = 0; p < P; ++p) next[p] = load_words<K>(bits[p] + (size_t)(ct + nw) * tile_words(K) + lane_words);
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const bool late = EITHER && beyond_fp16();
            if (late) left |= 1ull << min(2 * (ct / nw) + c, 63);
            else if (BF16 && !EITHER) put_wide();
            else put();
            if (c == 0) request(ct * TILE_COLS + UNIT_COLS);
            else if (ct + nw < CT) request((ct + nw) * TILE_COLS);
            if (!late) contract(std::integral_constant<int, BF16 && !EITHER ? 2 : 1>(), c);
            __builtin_amdgcn_wave_barrier();
        }
        if (AHEAD) {
#pragma unroll
            for (int p = 0; p < P; ++p) w[p] = next[p];
        } else if (ct + nw < CT) {
#pragma unroll
            for (int p = 0; p < P; ++p) w[p] = load_words<K>(bits[p] + (size_t)(ct + nw) * tile_words(K) + lane_words);
        }
    }
    if (EITHER && left != 0)                                   // (a bit too many costs a second look)
#pragma unroll 1
        for (int ct = wave; ct < CT; ct += nw) {
            if (!(left >> min(2 * (ct / nw), 62) & 3)) continue;
#pragma unroll
            for (int p = 0; p < P; ++p) w[p] = load_words<K>(bits[p] + (size_t)ct * tile_words(K) + lane_words);
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                request(ct * TILE_COLS + c * UNIT_COLS);
                if (!beyond_fp16()) continue;
                put_wide();
                contract(std::integral_constant<int, 2>(), c);
                __builtin_amdgcn_wave_barrier();
            }
        }
#pragma unroll
    for (int i = 0; i < GV; ++i) {
        const int at = tid + i * (int)blockDim.x;
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
    for (int idx = tid; idx < P * G * 256; idx += (int)blockDim.x) {
        const int p = idx / (G * 256), t = idx / 16 % (G * 16), row = (rt0 + p) * TILE_ROWS + idx % 16;
        float s = 0.f;
        for (int v = 0; v < nw; ++v) s += part[v * (P * G * 256) + idx];
        if (t < T && row < out) store_out(op.y, args.out_dtype, (size_t)t * out + row, s);
    }
}

// ------------------------------------------------------------------ host ---
constexpr int ROW_TILES_PER_WG[] = {1, 2, 3, 4, 6};

// Row tiles per workgroup: the device runs the workgroups in rounds of one per compute unit; a
// round takes as long as its row tiles plus what every workgroup pays once (reading the
// activations, the latencies, the sum), about one and a half row tiles' worth
static int row_tiles_per_wg(const int *RT, int nops, int K, int G)
{
    const int cus = std::max(1, mx::device_groups());
    int best = 1;
    double best_cost = 0.0;
    for (int P : ROW_TILES_PER_WG) {
        if (!p_available(K, G, P)) continue;
        int groups = 0;
        for (int i = 0; i < nops; ++i) groups += (RT[i] + P - 1) / P;
        const double cost = (double)((groups + cus - 1) / cus) * (P + 1.5);
        if (P == 1 || cost < best_cost) { best = P; best_cost = cost; }
    }
    return best;
}

template <int K, int G, int P, bool BF16>
static int launch_form(const Args &args, int groups, int nw, hipStream_t stream)
{
    constexpr int per_wave = std::max(slab_bytes<K, G, BF16>(), P * G * 1024), lds_max = max_waves(K, G, P) * per_wave;
    if (lds_max + P * K * TILE_ROWS * (int)sizeof(float) > 64 * 1024) {
        static std::atomic<bool> allowed[64];
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return RB_ERR_HIP;
        if (!allowed[dev].load()) {
            if (hipFuncSetAttribute(reinterpret_cast<const void *>(batch_kernel<K, G, P, BF16>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    lds_max) != hipSuccess)
                return RB_ERR_HIP;
            allowed[dev].store(true);
        }
    }
    hipLaunchKernelGGL((batch_kernel<K, G, P, BF16>), dim3((unsigned)groups), dim3((unsigned)(nw * 64)), nw * per_wave, stream, args);
    return RB_OK;
}

template <int K, int G, bool BF16>
static int launch_p(const Args &args, int P, int groups, int nw, hipStream_t stream)
{
    switch (P) {
    case 1: return launch_form<K, G, 1, BF16>(args, groups, nw, stream);
    case 2: if constexpr (p_available(K, G, 2)) return launch_form<K, G, 2, BF16>(args, groups, nw, stream); break;
    case 3: if constexpr (p_available(K, G, 3)) return launch_form<K, G, 3, BF16>(args, groups, nw, stream); break;
    case 4: if constexpr (p_available(K, G, 4)) return launch_form<K, G, 4, BF16>(args, groups, nw, stream); break;
    default: if constexpr (p_available(K, G, 6)) return launch_form<K, G, 6, BF16>(args, groups, nw, stream); break;
    }
    return RB_ERR_UNSUPPORTED;
}

static int token_groups(int T) { return T <= 16 ? 1 : T <= 32 ? 2 : 4; }

// one launch: the ops of `args` (wg0 is filled in here), all of K paths
struct Shape { int K, P, groups, nw; };
static Shape shape_of(Args &args, int K)
{
    int RT[MAX_STAGE_OPS], CT = 1;
    for (int i = 0; i < args.nops; ++i) {
        RT[i] = row_tiles(args.op[i].out);
        CT = std::max(CT, col_tiles(args.op[i].in));
    }
    Shape s;
    s.K = K;
    const int G = token_groups(args.T);
    s.P = row_tiles_per_wg(RT, args.nops, K, G);
    s.groups = 0;
    for (int i = 0; i < MAX_STAGE_OPS; ++i) {
        args.wg0[i] = i < args.nops ? s.groups : INT_MAX;
        if (i < args.nops) s.groups += (RT[i] + s.P - 1) / s.P;
    }
    s.nw = std::min(CT, max_waves(K, G, s.P));      // a wavefront takes whole column tiles
    return s;
}

template <bool BF16> static int launch_shape(const Args &args, const Shape &s, hipStream_t stream)
{
    const int G = token_groups(args.T);
    if (s.K == 2)
        return G == 1 ? launch_p<2, 1, BF16>(args, s.P, s.groups, s.nw, stream)
             : G == 2 ? launch_p<2, 2, BF16>(args, s.P, s.groups, s.nw, stream)
                      : launch_p<2, 4, BF16>(args, s.P, s.groups, s.nw, stream);
    return G == 1 ? launch_p<3, 1, BF16>(args, s.P, s.groups, s.nw, stream)
         : G == 2 ? launch_p<3, 2, BF16>(args, s.P, s.groups, s.nw, stream)
                  : launch_p<3, 4, BF16>(args, s.P, s.groups, s.nw, stream);
}

static Op make_op(const rb_layer &L, const void *x, void *y)
{
    Op o;
    o.bits = static_cast<const uint32_t *>(L.bits);
    o.g = L.g; o.h = L.h;
    o.x = x; o.y = y;
    o.out = L.out; o.in = L.in;
    o.h_aligned = ((uintptr_t)L.h & 15) == 0; o.pad_ = 0;
    return o;
}

// (the kernel keeps 32-bit offsets into the input)
static bool supported(const rb_layer *L, int T, int max_T)
{
    return (L->K == 2 || L->K == 3) && T >= 1 && T <= max_T && L->in % 32 == 0 && (size_t)T * L->in < (size_t)1 << 32;
}

bool call_supported(const rb_layer *L, int T) { return supported(L, T, CALL_MAX_T); }

int launch_call(const rb_layer *L, const void *X, void *Y, int T, int act_dtype, int out_dtype, void *workspace,
                size_t workspace_bytes, hipStream_t stream)
{
    // (one and two tokens: nothing is asked for, and the output must not overlap the input)
    if (T > 2 && overlap(X, input_bytes(L, T), Y, output_bytes(L, T, out_dtype))) {
        if (!workspace || workspace_bytes < aside_bytes(L, T)) return RB_ERR_WORKSPACE;
        copy_aside(X, workspace, input_bytes(L, T), stream);
        X = workspace;
    }
    Args args = {};
    args.nops = 1; args.T = T; args.out_dtype = out_dtype;
    args.op[0] = make_op(*L, X, Y);
    const Shape s = shape_of(args, L->K);
    const int rc = act_dtype == RB_BF16 ? launch_shape<true>(args, s, stream) : launch_shape<false>(args, s, stream);
    if (rc != RB_OK) return rc;
    return hipGetLastError() == hipSuccess ? RB_OK : RB_ERR_HIP;
}

bool layer_supported(const rb_layer *L, int T) { return supported(L, T, STACK_MAX_T); }

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
        args.nops = 0; args.T = T; args.out_dtype = RB_F16;
        const int K = layers[sops[op0].layer].K;
        for (int n = op0; n < n_ops && args.nops < MAX_STAGE_OPS; ++n) {
            const rb_layer &L = layers[sops[n].layer];
            bool conflict = L.K != K || (n > op0 && (meet(src(n), dst(n)) || meet(src(op0), dst(op0))));
            for (int m = op0; m < n; ++m)
                if (meet(dst(m), src(n)) || meet(dst(m), dst(n)) || meet(src(m), dst(n))) conflict = true;
            if (conflict) break;
            args.op[args.nops++] = make_op(L, bufs[sops[n].src], bufs[sops[n].dst]);
        }
        const Shape shape = shape_of(args, K);                 // (numbers the workgroups in args)
        Launch l = {args, shape, nullptr, 0};
        if (meet(src(op0), dst(op0))) {
            l.aside = src(op0).at;
            l.aside_bytes = src(op0).bytes;
            l.args.op[0].x = workspace;
        }
        pr->launches.push_back(l);
        op0 += args.nops;
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
