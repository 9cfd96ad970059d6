// Training-side kernels of the residual-binary layer (Section 4.2, Alg. 2).
//
//   * rb_couple: the on-the-fly residual coupling of the forward pass.  From the shared
//     full-precision weight and the scales it derives the binary cores path after path,
//     B_i = sign(R_{i-1}), R_i = R_{i-1} - g_i (.) B_i (.) h_i, and writes them packed (canonical
//     words and/or the kernel-native tiles the inference kernels read), so that a training step
//     can run its forward pass through the same kernels as inference.
//   * rb_weight_grad: the effective-weight gradient G = (dL/dY) X^T (Eq. RaBiT-grad-wfp), the
//     straight-through gradient of the shared weight.
//   * rb_scale_grads: the gradients of the scales (Eq. RaBiT-grad-gh) with the binary cores held
//     constant.  Summed over the samples they are signed reductions of G:
//         grad g_i[r] = sum_c B_i[r][c] h_i[c] G[r][c]       (rows)
//         grad h_i[c] = sum_r B_i[r][c] g_i[r] G[r][c]       (columns: the transposed product)
//     so one pass over G per direction gives them for every path, whatever the batch size.
//
// The first and the last are bound by HBM (4 bytes per weight read); the weight gradient is a dense
// contraction on the matrix cores.  Every sum runs in a fixed order, so results do not depend on scheduling.
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>

#include <type_traits>

#include "rabit.h"
#include "rb_device.h"
#include "rb_internal.h"
#include "rb_layout.h"

namespace rb {
namespace train {

constexpr int ROW_SLICE = 64;          // rows one workgroup of the column reduction walks
constexpr int COUPLE_CHUNK = 512, COUPLE_ROWS = 4;      // columns and rows one wavefront of the coupling kernel takes

// ------------------------------------------------------------------ couple ---
// A workgroup takes one row tile (16 rows, four wavefronts of COUPLE_ROWS) and COUPLE_CHUNK columns: its native tiles are put
// together in LDS and stored in whole lines, padding included (zero bits: +1).  What a wavefront's rows share of
// the columns (h, converted to fp32) is fetched once.  A lane takes four consecutive columns
// at a time (one 16-byte load of W; the chunk's loads are all requested before the first is used),
// so a step of the wavefront covers 256 columns.  The comparison of column j of the lanes is a 64-bit
// mask in scalar registers whose bits 8 w .. 8 w + 7 belong to sign word w of the step; its halves
// are filed in lanes of a register of their own for each j, and at the end 64 lanes put 64 words
// together at once: lane (step, row, w) fetches its byte of the four masks (bit 8 j + i is column 4 i + j)
// and moves the bits to where the canonical word (bit 4 i + j) and the native one (native bit 4 e + s is
// column 8 s + e: bit 16 (i % 2) + 4 j + i / 2) have them.
// The residual is fp32 with one rounding for g * h and one for
// the subtraction, the arithmetic the definition fixes (the sign of the product is exact).
// Bound by the read of W and, behind it, by vector instructions.
// Vector instructions of a wavefront at two paths 500, with an OR over eight lanes per word and form and h fetched where it was used
// 877; a training step of 4096 x 11008 (512 samples) 228.6 -> 223.3 us by this alone.  (The words by themselves before that, one row per
// wavefront and native words stored one by one: 8 us more, and 6 for zeroing them before.)
extern "C" __device__ uint32_t rb_writelane(uint32_t value, uint32_t lane, uint32_t old) __asm("llvm.amdgcn.writelane.i32");      // has no builtin
template <int A, int B> __device__ __forceinline__ uint32_t swap_index_bits(uint32_t x)      // bit i of a word goes where bits A > B of i are exchanged
{
    constexpr int D = (1 << A) - (1 << B);
    constexpr uint32_t b[5] = {0xaaaaaaaau, 0xccccccccu, 0xf0f0f0f0u, 0xff00ff00u, 0xffff0000u}, mask = b[B] & ~b[A];
    const uint32_t t = (x ^ x >> D) & mask;
    return x ^ t ^ t << D;
}

template <int K>
__global__ __launch_bounds__(256) void couple_kernel(const float *__restrict__ W, const __half *__restrict__ g,
                                                     const __half *__restrict__ h, int out, int in,
                                                     uint32_t *__restrict__ packed, uint32_t *__restrict__ native,
                                                     float *__restrict__ residual)
{
    constexpr int STEPS = COUPLE_CHUNK / 256, R = COUPLE_ROWS;
    static_assert(STEPS * R * 8 == 64 && STEPS * K * R * 2 <= 64, "a path's words are a wavefront's lanes, the masks' halves fit them");
    const int lane = threadIdx.x & 63;
    // one-dimensional grid, row tiles fastest (a second dimension would end at 65536 chunks of columns)
    const int RT = row_tiles(out), rt = (int)(blockIdx.x % (unsigned)RT);
    const int tile_row0 = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6) * R), row0 = rt * TILE_ROWS + tile_row0;
    static_assert(4 * R == TILE_ROWS && COUPLE_CHUNK % TILE_COLS == 0, "whole sign tiles per workgroup");
    __shared__ __attribute__((aligned(16))) uint32_t tiles[STEPS * tile_words(K)];
    const int W32 = in / 32, CT = col_tiles(in);
    const int chunk0 = (int)(blockIdx.x / (unsigned)RT) * COUPLE_CHUNK;
    float4 wv[STEPS][R];
    uint2 hb[STEPS][K];
#pragma unroll
    for (int i = 0; i < STEPS; ++i) {
        const int c = chunk0 + 256 * i + 4 * lane;             // in % 32 == 0: all four columns or none
#pragma unroll
        for (int k = 0; k < K; ++k) hb[i][k] = *reinterpret_cast<const uint2 *>(h + (size_t)k * in + (c < in ? c : 0));
#pragma unroll
        for (int u = 0; u < R; ++u)                            // rows and columns past the end: others, whose signs `real` clears
            wv[i][u] = *reinterpret_cast<const float4 *>(W + (size_t)min(row0 + u, out - 1) * in + (c < in ? c : 0));
    }
    float gr[R][K];
#pragma unroll
    for (int u = 0; u < R; ++u)
#pragma unroll
        for (int k = 0; k < K; ++k) gr[u][k] = __half2float(g[(size_t)k * out + min(row0 + u, out - 1)]);
    uint32_t masks[4] = {0u, 0u, 0u, 0u};                      // column j: half v of (step i, path k, row u) in lane ((i K + k) R + u) 2 + v
#pragma unroll
    for (int i = 0; i < STEPS; ++i) {
        const int c = chunk0 + 256 * i + 4 * lane;
        const uint64_t real = __builtin_amdgcn_ballot_w64(c < in);
        float r[R][4];
#pragma unroll
        for (int u = 0; u < R; ++u) { r[u][0] = wv[i][u].x; r[u][1] = wv[i][u].y; r[u][2] = wv[i][u].z; r[u][3] = wv[i][u].w; }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const float hv[4] = {__half2float(__ushort_as_half((unsigned short)(hb[i][k].x & 0xffffu))),
                                 __half2float(__ushort_as_half((unsigned short)(hb[i][k].x >> 16))),
                                 __half2float(__ushort_as_half((unsigned short)(hb[i][k].y & 0xffffu))),
                                 __half2float(__ushort_as_half((unsigned short)(hb[i][k].y >> 16)))};
#pragma unroll
            for (int u = 0; u < R; ++u) {
                const uint64_t counts = row0 + u < out ? real : 0u;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const bool neg = !(r[u][j] >= 0.f);        // sign(0) = +1
                    const float prod = __fmul_rn(gr[u][k], hv[j]);
                    r[u][j] = __fsub_rn(r[u][j], neg ? -prod : prod);
                    const uint64_t m = __builtin_amdgcn_ballot_w64(neg) & counts;
                    const int at = ((i * K + k) * R + u) * 2;
                    masks[j] = rb_writelane((uint32_t)m, at, masks[j]);
                    masks[j] = rb_writelane((uint32_t)(m >> 32), at + 1, masks[j]);
                }
            }
        }
        if (residual && c < in)
#pragma unroll
            for (int u = 0; u < R; ++u)
                if (row0 + u < out) *reinterpret_cast<float4 *>(residual + (size_t)(row0 + u) * in + c) = make_float4(r[u][0], r[u][1], r[u][2], r[u][3]);
    }
    // this lane's word of each path: step, row, word of the step
    const int i = lane >> 5, u = lane >> 3 & 3, w = lane & 7;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int from = ((i * K + k) * R + u) * 2 + (w >> 2);
        uint32_t x = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            x |= ((uint32_t)__builtin_amdgcn_ds_bpermute(4 * from, (int)masks[j]) >> 8 * (w & 3) & 0xffu) << 8 * j;
        const int word = (chunk0 >> 5) + 8 * i + w;
        if (packed && word < W32 && row0 + u < out)            // index bits j j i i i -> i i i j j
            packed[((size_t)k * out + row0 + u) * W32 + word] =
                swap_index_bits<1, 0>(swap_index_bits<2, 0>(swap_index_bits<3, 1>(swap_index_bits<4, 2>(x))));
        tiles[i * tile_words(K) + lane_word(tile_row0 + u + 16 * (w & 3), w >> 2, k, K)] =      // j j i i i0 -> i0 j j i i
            swap_index_bits<1, 0>(swap_index_bits<2, 0>(swap_index_bits<3, 0>(swap_index_bits<4, 0>(x))));
    }
    if (!native) return;
    __syncthreads();
    const int ct0 = chunk0 / TILE_COLS, words = min(STEPS, CT - ct0) * tile_words(K);
    uint32_t *const dst = native + ((size_t)rt * CT + ct0) * tile_words(K);      // 4-byte aligned at least
    for (int i = threadIdx.x; i < words; i += 256) dst[i] = tiles[i];
}

// --------------------------------------------------------------- gradients ---
// G = Delta^T X (Eq. RaBiT-grad-wfp) on the matrix cores: fp16 operands, exact products, fp32 sums.
//
// Bound by the store of G (4 bytes per weight) up to a few hundred samples and by the matrix units
// beyond: one tile of WG_ROWS x WG_COLS outputs per workgroup, a wavefront owns 64 x 128 of it (2 x 4
// accumulators of 32 x 32), two workgroups share a compute unit so that one stores while the other
// multiplies.  Both operands lie in memory with the samples outermost while the matrix instruction
// wants eight consecutive samples per lane, so a thread loads a block of samples x 4 columns (8 bytes per
// sample, whole rows of a tile coalesced), transposes it in registers (one byte permute per dword)
// and writes one group of consecutive samples per column to LDS.  LDS holds [group of 8 samples][slot][8 samples]
// with the columns of a wavefront de-interleaved (slot 32 i + q holds column 4 q + i), so that
//   * a write covers consecutive slots (no bank conflicts), and so does an operand read;
//   * the four column accumulators of a lane are four consecutive columns of G: 16-byte stores.
// 4096 x 11008, calls in a row in a graph: 76 to 83 us from card to card at 512 samples (0.56 to 0.61 PFLOP/s, 2.2 TB/s of G stored), 223 to 229
// at 2048, 33 at 33; with one step in flight, its loads in branches and so every wait for all of them, 86 to 94, 261 to 269 and 33 to 35.  In
// a kernel trace 74.  The store of a tile and the multiplications of the next do not overlap
// much (33 us of the 76 are what 33 samples take): all workgroups run in step.
constexpr int WG_ROWS = 128, WG_COLS = 256, WG_N = 32;      // tile of G, samples per step
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

// four columns of one sample (zero past the end of the samples or the columns), two bytes at a time or (EIGHT) all at once
template <bool EIGHT> __device__ __forceinline__ uint2 load_cols(const __half *p, size_t n, size_t N, int c, int width)
{
    uint2 v = make_uint2(0u, 0u);
    if (n >= N) return v;
    const unsigned short *row = reinterpret_cast<const unsigned short *>(p) + (size_t)n * width;
    if (EIGHT) {
        if (c < width) v = *reinterpret_cast<const uint2 *>(row + c);
        return v;
    }
    if (c < width) v.x = row[c];
    if (c + 1 < width) v.x |= (uint32_t)row[c + 1] << 16;
    if (c + 2 < width) v.y = row[c + 2];
    if (c + 3 < width) v.y |= (uint32_t)row[c + 3] << 16;
    return v;
}
// loads that return zero past the end of their buffer (NOWHERE always is)
constexpr uint32_t NOWHERE = 0x40000000u;
constexpr int WG_MAX_WIDTH = 1 << 23;                       // WG_N rows of that many columns stay below NOWHERE
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer(const void *p, size_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ uint32_t low_halves(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x05040100u); }
__device__ __forceinline__ uint32_t high_halves(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }

// FORM: rows of Delta, X and G that start at multiples of 8 (G: 16) bytes (ALIGNED), of X and G only (DELTA_OFF: Delta's are read
// as they lie; 4095 x 4096 with 512 samples 35 us, 115 two bytes at a time), neither (ANY: two bytes at a time).  WIDE: ALIGNED, but from WG_MAX_WIDTH columns on, beyond the offsets of a buffer:
// 8-byte loads in branches, one step in flight (132 x 2^23 with 96 samples 1.7 ms, 4.7 two bytes at a time)
enum Form { ALIGNED, DELTA_OFF, WIDE, ANY };
template <Form FORM>
__global__ __launch_bounds__(256, 2) void weight_grad_kernel(const __half *__restrict__ Delta, const __half *__restrict__ X,
                                                             int N, int out, int in, float *__restrict__ G)
{
    constexpr bool VEC = FORM == ALIGNED || FORM == DELTA_OFF;
    constexpr int A_BYTES = WG_ROWS * WG_N * 2, B_BYTES = WG_COLS * WG_N * 2;
    __shared__ __attribute__((aligned(16))) uint8_t lds[2][A_BYTES + B_BYTES];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wr = wave >> 1, wc = wave & 1;
    // workgroups go round the eight XCDs: each takes a run of tiles, row tiles fastest, so that one
    // block of columns of X and all of Delta (N x out) are what its L2 sees
    const int tiles_r = (out + WG_ROWS - 1) / WG_ROWS, tiles = tiles_r * ((in + WG_COLS - 1) / WG_COLS);
    const int per = (tiles + 7) / 8, tile = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per || tile >= tiles) return;
    const int r0 = tile % tiles_r * WG_ROWS, c0 = tile / tiles_r * WG_COLS;

    // this thread's part of a step: 4 samples x 4 columns of Delta, 8 samples x 4 columns of X
    const int qa = tid & 31, na = tid >> 5, qb = tid & 63, nb = tid >> 6;
    const int slot_a = (qa >> 4) * 64 + (qa & 15), slot_b = (qb >> 5) * 128 + (qb & 31);
    // Two steps are in flight beside the one that is multiplied: a step is 0.5 us of matrix instructions, less than its loads take.  They
    // sit in buffers of their own (set 0, 1), and no branch is around any of them
    constexpr int SETS = VEC ? 2 : 1;
    uint2 da[SETS][4], xb[SETS][8];
    const uint32_t a_off = r0 + 4 * qa < out ? ((uint32_t)(4 * na) * (uint32_t)out + (uint32_t)(r0 + 4 * qa)) * 2u : NOWHERE;
    // Delta off alignment: the four columns from a_at, moved down by a_shift bits where those are not the lane's own
    const uint32_t a_at = (uint32_t)min(r0 + 4 * qa, out - 4), a_shift = 16u * (uint32_t)min(r0 + 4 * qa - (int)a_at, 4);
    const uint32_t b_off = c0 + 4 * qb < in ? ((uint32_t)(8 * nb) * (uint32_t)in + (uint32_t)(c0 + 4 * qb)) * 2u : NOWHERE;
    auto request = [&](size_t n0, auto set) {
        if constexpr (VEC) {
            const size_t rows = min((size_t)WG_N, (size_t)N - n0);
            const __amdgpu_buffer_rsrc_t a_rs = buffer(Delta + n0 * out, rows * out * 2), b_rs = buffer(X + n0 * in, rows * in * 2);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (FORM == ALIGNED) da[set][j] = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(a_rs, (int)(a_off + (uint32_t)j * (uint32_t)out * 2u), 0, 0));
                // (samples past the end: the last one, whose X reads as zero and which `put` clears)
                else __builtin_memcpy(&da[set][j], Delta + n0 * out + (size_t)((uint32_t)min(4 * na + j, (int)rows - 1) * (uint32_t)out + a_at), 8);
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) xb[set][j] = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(b_rs, (int)(b_off + (uint32_t)j * (uint32_t)in * 2u), 0, 0));
            __builtin_amdgcn_sched_barrier(0);
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) da[set][j] = load_cols<FORM == WIDE>(Delta, n0 + 4 * na + j, N, r0 + 4 * qa, out);
#pragma unroll
            for (int j = 0; j < 8; ++j) xb[set][j] = load_cols<FORM == WIDE>(X, n0 + 8 * nb + j, N, c0 + 4 * qb, in);
        }
    };
    auto put = [&](uint8_t *buf, auto set, [[maybe_unused]] size_t n0) {
        uint2 d[4];
        const uint2 (&x)[8] = xb[set];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            d[j] = da[set][j];
            if (FORM == DELTA_OFF) {
                const unsigned long long v = __builtin_bit_cast(unsigned long long, d[j]);
                d[j] = __builtin_bit_cast(uint2, a_shift < 64 && n0 + 4 * na + j < (size_t)N ? v >> a_shift : 0ull);
            }
        }
        uint8_t *const a = buf + (na >> 1) * (WG_ROWS * 16) + slot_a * 16 + (na & 1) * 8;
        *reinterpret_cast<uint2 *>(a) = make_uint2(low_halves(d[0].x, d[1].x), low_halves(d[2].x, d[3].x));
        *reinterpret_cast<uint2 *>(a + 16 * 16) = make_uint2(high_halves(d[0].x, d[1].x), high_halves(d[2].x, d[3].x));
        *reinterpret_cast<uint2 *>(a + 32 * 16) = make_uint2(low_halves(d[0].y, d[1].y), low_halves(d[2].y, d[3].y));
        *reinterpret_cast<uint2 *>(a + 48 * 16) = make_uint2(high_halves(d[0].y, d[1].y), high_halves(d[2].y, d[3].y));
        uint8_t *const b = buf + A_BYTES + nb * (WG_COLS * 16) + slot_b * 16;
        uint4 v[4];
        uint32_t *const w = reinterpret_cast<uint32_t *>(v);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            w[j] = low_halves(x[2 * j].x, x[2 * j + 1].x);
            w[4 + j] = high_halves(x[2 * j].x, x[2 * j + 1].x);
            w[8 + j] = low_halves(x[2 * j].y, x[2 * j + 1].y);
            w[12 + j] = high_halves(x[2 * j].y, x[2 * j + 1].y);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) *reinterpret_cast<uint4 *>(b + i * 32 * 16) = v[i];
    };

    v16f acc[2][4];
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[m][i][e] = 0.f;

    auto multiply = [&](const uint8_t *buf) {
        const uint8_t *const a = buf + (wr * 64 + (lane & 31)) * 16, *const b = buf + A_BYTES + (wc * 128 + (lane & 31)) * 16;
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            const int group = 2 * kk + (lane >> 5);
            v8h av[2], bv[4];
#pragma unroll
            for (int m = 0; m < 2; ++m) av[m] = *reinterpret_cast<const v8h *>(a + group * (WG_ROWS * 16) + m * 32 * 16);
#pragma unroll
            for (int i = 0; i < 4; ++i) bv[i] = *reinterpret_cast<const v8h *>(b + group * (WG_COLS * 16) + i * 32 * 16);
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[m][i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(av[m], bv[i], acc[m][i], 0, 0, 0);
        }
    };
    constexpr std::integral_constant<int, 0> S0;
    constexpr std::integral_constant<int, SETS - 1> S1;
    // (sample numbers in 64 bits: beyond 2^31 - 128 of them the next steps' would not be an int)
    request(0, S0);
    if constexpr (VEC) {
        // (the last steps by themselves: a request that fetches nothing takes its turn all the same, and one in a branch would make
        // every wait as long as the longest)
        const size_t steps = ((size_t)N + WG_N - 1) / WG_N;
        if (steps > 1) request(WG_N, S1);
        put(lds[0], S0, 0);
        if (steps > 2) request(2 * WG_N, S0);
        size_t s = 0;
        for (; s + 4 < steps; s += 2) {
            __syncthreads();                               // this step's tile is complete, the other one free
            multiply(lds[0]);
            put(lds[1], S1, (s + 1) * WG_N);
            request((s + 3) * WG_N, S1);
            __syncthreads();
            multiply(lds[1]);
            put(lds[0], S0, (s + 2) * WG_N);
            request((s + 4) * WG_N, S0);
        }
        __syncthreads();
        multiply(lds[0]);
        if (s + 1 < steps) {
            put(lds[1], S1, (s + 1) * WG_N);
            if (s + 3 < steps) request((s + 3) * WG_N, S1);
            __syncthreads();
            multiply(lds[1]);
        }
        if (s + 2 < steps) {
            put(lds[0], S0, (s + 2) * WG_N);
            __syncthreads();
            multiply(lds[0]);
        }
        if (s + 3 < steps) {
            put(lds[1], S1, (s + 3) * WG_N);
            __syncthreads();
            multiply(lds[1]);
        }
    } else {
        put(lds[0], S0, 0);
        int cur = 0;
        for (size_t n0 = 0; n0 < (size_t)N; n0 += WG_N, cur ^= 1) {
            const bool more = n0 + WG_N < (size_t)N;
            if (more) request(n0 + WG_N, S0);
            __syncthreads();
            multiply(lds[cur]);
            if (more) put(lds[cur ^ 1], S0, n0 + WG_N);
        }
    }

    // accumulator element e of a lane: matrix row rho = 8 (e / 4) + 4 (lane / 32) + e % 4, column lane % 32;
    // row block m holds row 4 (rho % 16) + 2 m + rho / 16 of the wavefront's 64
    const int c = c0 + wc * 128 + 4 * (lane & 31);
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int rho = 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
            const int r = r0 + wr * 64 + 4 * (rho & 15) + 2 * m + (rho >> 4);
            if (r >= out) continue;
            float *const dst = G + (size_t)r * in + c;
            if (FORM != ANY) {
                if (c < in) *reinterpret_cast<float4 *>(dst) = make_float4(acc[m][0][e], acc[m][1][e], acc[m][2][e], acc[m][3][e]);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (c + i < in) dst[i] = acc[m][i][e];
            }
        }
}

// Both scale gradients from one pass over G (4096 x 11008, two paths: 36 us + 4.5 for the sums; 43 with the paths counted at run time, a
// conversion of all three paths' h and loads in branches; with the next eight rows in flight as well, which spills, 51).  A wavefront takes a slab of ROW_SLICE rows by 256
// columns, a lane four consecutive columns (one 16-byte load of G and four bits of a sign word per
// row and path), eight rows in flight.  The column sums of grad h stay in the lane (rows in order);
// the row sums of grad g need the whole wavefront: the eight rows of a group are summed together,
// three exchanges that each halve the number of rows a lane carries (after them lane l holds row
// 4 (l & 1) + 2 (l >> 1 & 1) + (l >> 2 & 1) of the group, summed over its eight lanes) and three
// more over the eight-lane groups.  Partial sums: [slice][K][in] and [column block][K][out]; the
// second kernel adds them in order, so results repeat bit for bit.
template <int K>
__global__ __launch_bounds__(64, K < 3 ? 4 : 2) void grad_slab_kernel(const float *__restrict__ G, const uint32_t *__restrict__ packed,
                                                          const __half *__restrict__ g, const __half *__restrict__ h,
                                                          int out, int in, float *__restrict__ part_h,
                                                          float *__restrict__ part_g)
{
    const int lane = threadIdx.x;
    const int c = (blockIdx.x * 64 + lane) * 4, slice = blockIdx.y;
    const bool real = c < in;                                  // in % 32 == 0: all four columns or none
    const int cs = real ? c : 0;
    const int W32 = in / 32, r0 = slice * ROW_SLICE, r1 = min(out, r0 + ROW_SLICE);
    // eight rows: no branch around their loads (rows past the end: the last one, whose values do not count)
    struct Rows { float4 v[8]; uint32_t bits[K][8]; };
    auto fetch = [&](int rb, Rows &to) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int r = min(rb + u, r1 - 1);
            to.v[u] = *reinterpret_cast<const float4 *>(G + (size_t)r * in + cs);
#pragma unroll
            for (int k = 0; k < K; ++k) to.bits[k][u] = packed[((size_t)k * out + r) * W32 + (cs >> 5)];
        }
    };
    float sh[K][4], hv[K][4];
#pragma unroll
    for (int k = 0; k < K; ++k) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float f = __half2float(h[(size_t)k * in + cs + e]);
            hv[k][e] = real ? f : 0.f;                         // (a lane past the end adds nothing, also where f is infinite)
            sh[k][e] = 0.f;
        }
    }
    const bool b0 = lane & 1, b1 = lane & 2, b2 = lane & 4;
    const int my_row = 4 * (int)b0 + 2 * (int)b1 + (int)b2;
#pragma unroll 1
    for (int rb = r0; rb < r1; rb += 8) {
        Rows now;
        fetch(rb, now);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            float rp[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const bool counts = real && rb + u < r1;
                const float v[4] = {counts ? now.v[u].x : 0.f, counts ? now.v[u].y : 0.f, counts ? now.v[u].z : 0.f, counts ? now.v[u].w : 0.f};
                const uint32_t bits4 = now.bits[k][u] >> (cs & 31);
                const float gk = __half2float(g[(size_t)k * out + min(rb + u, r1 - 1)]);
                float rs = 0.f;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float sv = __uint_as_float(__float_as_uint(v[e]) ^ (bits4 << (31 - e) & 0x80000000u));
                    sh[k][e] = __builtin_fmaf(gk, sv, sh[k][e]);
                    rs = __builtin_fmaf(hv[k][e], sv, rs);
                }
                rp[u] = rs;
            }
            float q[4], p2[2];
#pragma unroll
            for (int u = 0; u < 4; ++u) q[u] = (b0 ? rp[u + 4] : rp[u]) + __shfl_xor(b0 ? rp[u] : rp[u + 4], 1);
#pragma unroll
            for (int u = 0; u < 2; ++u) p2[u] = (b1 ? q[u + 2] : q[u]) + __shfl_xor(b1 ? q[u] : q[u + 2], 2);
            float o = (b2 ? p2[1] : p2[0]) + __shfl_xor(b2 ? p2[0] : p2[1], 4);
            o += __shfl_xor(o, 8);
            o += __shfl_xor(o, 16);
            o += __shfl_xor(o, 32);
            if (lane < 8 && rb + my_row < r1) part_g[((size_t)blockIdx.x * K + k) * out + rb + my_row] = o;
        }
    }
    if (real)
#pragma unroll
        for (int k = 0; k < K; ++k)
            *reinterpret_cast<float4 *>(part_h + ((size_t)slice * K + k) * in + c) =
                make_float4(sh[k][0], sh[k][1], sh[k][2], sh[k][3]);
}

// element i < K * in of grad h: the slices in order; the rest, grad g: the column blocks in order
__global__ __launch_bounds__(256) void grad_finish_kernel(const float *__restrict__ part_h, int slices,
                                                          const float *__restrict__ part_g, int col_blocks, int K,
                                                          int out, int in, float *__restrict__ grad_g,
                                                          float *__restrict__ grad_h)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < K * in) {
        float s = 0.f;
#pragma unroll 8
        for (int sl = 0; sl < slices; ++sl) s += part_h[(size_t)sl * K * in + i];
        grad_h[i] = s;
    } else if (i < K * in + K * out) {
        const int j = i - K * in;
        float s = 0.f;
#pragma unroll 8
        for (int cb = 0; cb < col_blocks; ++cb) s += part_g[(size_t)cb * K * out + j];
        grad_g[j] = s;
    }
}

static int check_shape(int K, int out, int in)
{
    return (K < 1 || K > RB_MAX_K || out < 1 || in < 32 || in % 32 != 0) ? RB_ERR_SHAPE : RB_OK;
}

}  // namespace train
}  // namespace rb

using namespace rb::train;

extern "C" int rb_couple(const float *W, const uint16_t *g, const uint16_t *h, int K, int out, int in,
                         uint32_t *packed, void *native, float *residual, void *stream_)
{
    if (!W || !g || !h) return RB_ERR_NULL;
    if (!packed && !native) return RB_ERR_NULL;
    const int rc = check_shape(K, out, in);
    if (rc != RB_OK) return rc;
    if (((uintptr_t)packed | (uintptr_t)native) & 3) return RB_ERR_ALIGN;
    if (((uintptr_t)W | (uintptr_t)residual) & 15) return RB_ERR_ALIGN;
    if ((uintptr_t)h & 7) return RB_ERR_ALIGN;
    hipStream_t stream = static_cast<hipStream_t>(stream_);
    const dim3 grid((unsigned)rb::row_tiles(out) * (((unsigned)in + COUPLE_CHUNK - 1) / COUPLE_CHUNK));
    auto run = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(256), 0, stream, W, reinterpret_cast<const __half *>(g),
                           reinterpret_cast<const __half *>(h), out, in, packed, static_cast<uint32_t *>(native), residual);
    };
    if (K == 1) run(couple_kernel<1>);
    else if (K == 2) run(couple_kernel<2>);
    else run(couple_kernel<3>);
    return hipGetLastError() == hipSuccess ? RB_OK : RB_ERR_HIP;
}

extern "C" int rb_weight_grad(const uint16_t *Delta, const uint16_t *X, int N, int out, int in, float *G, void *stream_)
{
    if (!Delta || !X || !G) return RB_ERR_NULL;
    if (N < 1 || out < 1 || in < 1 || out > 65535) return RB_ERR_SHAPE;
    const int tiles = (out + WG_ROWS - 1) / WG_ROWS * ((in + WG_COLS - 1) / WG_COLS);
    const dim3 grid((unsigned)((tiles + 7) / 8 * 8));
    const bool x_aligned = in % 4 == 0 && ((uintptr_t)X & 7) == 0 && ((uintptr_t)G & 15) == 0;
    const bool d_aligned = out % 4 == 0 && ((uintptr_t)Delta & 7) == 0;
    const __half *d = reinterpret_cast<const __half *>(Delta), *x = reinterpret_cast<const __half *>(X);
    hipStream_t stream = static_cast<hipStream_t>(stream_);
    auto run = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(256), 0, stream, d, x, N, out, in, G); };
    const bool fits = in < WG_MAX_WIDTH;
    if (x_aligned && d_aligned) fits ? run(weight_grad_kernel<ALIGNED>) : run(weight_grad_kernel<WIDE>);
    else if (x_aligned && out >= 4 && fits) run(weight_grad_kernel<DELTA_OFF>);
    else run(weight_grad_kernel<ANY>);
    return hipGetLastError() == hipSuccess ? RB_OK : RB_ERR_HIP;
}

extern "C" size_t rb_scale_grads_workspace_bytes(int K, int out, int in)
{
    if (check_shape(K, out, in) != RB_OK) return 0;
    // [slice][K][in] partial sums of grad h, then [column block][K][out] partial sums of grad g
    return ((size_t)((out + ROW_SLICE - 1) / ROW_SLICE) * K * in + (size_t)((in + 255) / 256) * K * out) * sizeof(float);
}

extern "C" int rb_scale_grads(const float *G, const uint32_t *packed, const uint16_t *g, const uint16_t *h, int K,
                              int out, int in, float *grad_g, float *grad_h, void *workspace, size_t workspace_bytes,
                              void *stream_)
{
    if (!G || !packed || !g || !h || !grad_g || !grad_h) return RB_ERR_NULL;
    const int rc = check_shape(K, out, in);
    if (rc != RB_OK) return rc;
    const int slices = (out + ROW_SLICE - 1) / ROW_SLICE;
    if (slices > 65535) return RB_ERR_SHAPE;
    if (!workspace || workspace_bytes < rb_scale_grads_workspace_bytes(K, out, in)) return RB_ERR_WORKSPACE;
    if (((uintptr_t)workspace | (uintptr_t)G) & 15) return RB_ERR_ALIGN;
    hipStream_t stream = static_cast<hipStream_t>(stream_);
    const int col_blocks = (in + 255) / 256;
    float *part_h = static_cast<float *>(workspace), *part_g = part_h + (size_t)slices * K * in;
    auto run = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)col_blocks, (unsigned)slices), dim3(64), 0, stream, G, packed,
                           reinterpret_cast<const __half *>(g), reinterpret_cast<const __half *>(h), out, in, part_h, part_g);
    };
    if (K == 1) run(grad_slab_kernel<1>);
    else if (K == 2) run(grad_slab_kernel<2>);
    else run(grad_slab_kernel<3>);
    hipLaunchKernelGGL(grad_finish_kernel, dim3((unsigned)((K * (in + out) + 255) / 256)), dim3(256), 0, stream, part_h,
                       slices, part_g, col_blocks, K, out, in, grad_g, grad_h);
    return hipGetLastError() == hipSuccess ? RB_OK : RB_ERR_HIP;
}
