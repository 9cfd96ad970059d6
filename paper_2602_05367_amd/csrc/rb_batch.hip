// Few-token kernel of the residual-binary layer: single calls and stacks of a handful to a few dozen
// tokens, two or three paths.  Every op streams its packed weights ONCE for all tokens.
//
// Section 4.1: Y[t] = sum_k g_k (.) (B_k (h_k (.) X[t])), here with the input scale on the side of the
// signs: the left operand of v_mfma_f32_16x16x32_f16 is +-h_k[j] (the stored fp16 scale with the sign
// bit of the weight put in), the right operand is the fp16 activation itself.  Both are exact, so are
// their products, and only fp32 sums round; the activation is shared by the paths, nothing about the
// input is prepared, and an op is one launch.  What bounds it:
//   * a launch of a 4096-wide op moves 4 MB of signs, half a microsecond of HBM time, so it is a
//     chain of latencies (launch, one trip to memory, the matrix instructions, the sum over the
//     wavefronts): the compute units are filled and every wavefront asks for all it needs at once;
//   * beyond that, vector instructions: three per two weights and path (a byte permute that brings
//     two sign bits to bits 15 and 31, one three-input logic operation that puts them on the scales,
//     and a share of the shifts), 0.7 to 0.9 k clocks per 16 x 256 tile and SIMD, where the matrix
//     instructions of 16 tokens take 0.26 k.
// Shape: a workgroup owns P row tiles (16 rows) and all columns; its up to sixteen wavefronts share out the
// column tiles, each takes all P row tiles of its columns, so an activation is read from memory by
// one wavefront of the workgroup.  The partial outputs of the wavefronts meet in LDS and are added in
// a fixed order.  Nothing is exchanged between workgroups: no counters, no scratch memory, results do
// not depend on scheduling.  The ops of a stack that do not depend on each other (q/k/v, gate/up of
// a transformer block) run in one launch; dependent ones are ordered by the stream.
//
// Measured (start: bf8 term expansions staged in LDS with a ring of copies, a set-up launch per input,
// four launches for a single call): 7B-shaped dependent chain, 128 launches, 2.51 -> 1.42 ms at 8
// tokens and 3.09 -> 1.61 ms at 16; a launch takes 7.5 us (4096 x 4096, one row tile per workgroup) to 17 us
// (2 x 11008 x 4096, six), of which a dependent launch by itself is 4.7.  Single calls: 4096 x 11008
// with three paths at 16 tokens 107 -> 17 us, 10999 x 4128 with two at 7 tokens 42 -> 13 us.
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>

#include <algorithm>
#include <atomic>
#include <map>
#include <memory>
#include <mutex>
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

constexpr int STACK_MAX_T = 16;        // tokens of a stack
constexpr int MAX_STAGE_OPS = 8;       // independent ops that share a launch

// Wavefronts of a workgroup at most, and row tiles per workgroup: accumulators take 4 P K G
// registers and the activations of a column tile up to 32 G, of 128 with sixteen wavefronts per compute unit
// and 256 with eight
__host__ __device__ constexpr int max_waves(int G) { return G <= 2 ? 16 : 8; }
__host__ __device__ constexpr bool p_available(int K, int G, int P) { return P == 1 || P * K <= (G == 1 ? 12 : 6); }

struct Op {
    const uint32_t *bits;     // native sign tiles
    const uint16_t *g;        // fp16 [K][out]
    const uint16_t *h;        // fp16 [K][in]
    const void *x;            // [T][in]
    void *y;                  // [T][out]
    int out, in;
    int wg0;                  // first workgroup of this op inside its launch
    int h_even;               // h starts at a multiple of four bytes
};
// everything a launch needs, passed by value: no table in memory to fetch before the work starts
struct Args {
    Op op[MAX_STAGE_OPS];
    int nops, T, out_dtype;
};

// ------------------------------------------------------------------- kernel ---
// lane N of each row of 16 lanes, in all 16
template <int N> __device__ __forceinline__ uint32_t row_lane(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x150 + N, 0xf, 0xf, true);
}
__device__ __forceinline__ uint32_t row_lane(uint32_t v, int n)      // n: constant once the loop around the call is unrolled
{
    switch (n) {
    case 0: return row_lane<0>(v);
    case 1: return row_lane<1>(v);
    case 2: return row_lane<2>(v);
    case 3: return row_lane<3>(v);
    case 4: return row_lane<4>(v);
    case 5: return row_lane<5>(v);
    case 6: return row_lane<6>(v);
    case 7: return row_lane<7>(v);
    case 8: return row_lane<8>(v);
    case 9: return row_lane<9>(v);
    case 10: return row_lane<10>(v);
    case 11: return row_lane<11>(v);
    case 12: return row_lane<12>(v);
    case 13: return row_lane<13>(v);
    case 14: return row_lane<14>(v);
    default: return row_lane<15>(v);
    }
}

// two bf16 activations as a pair of fp16 values, halved: a bf16 value up to 1.3e5 stays finite, and the
// result is doubled again in fp32
__device__ __forceinline__ uint32_t half_of_bf16_pair(uint32_t v)
{
    const _Float16 lo = (_Float16)(0.5f * __uint_as_float(v << 16)), hi = (_Float16)(0.5f * __uint_as_float(v & 0xffff0000u));
    return (uint32_t)__builtin_bit_cast(unsigned short, lo) | ((uint32_t)__builtin_bit_cast(unsigned short, hi) << 16);
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

// K paths, G groups of 16 tokens, P row tiles per workgroup, BF16: the activations are bfloat16
template <int K, int G, int P, bool BF16>
__global__ __launch_bounds__(max_waves(G) * 64, 1) void batch_kernel(const Args args)
{
    constexpr bool AHEAD = P * K <= (G == 1 ? 6 : 4) && G <= 2;       // registers for the sign words of the next column tile
    constexpr int XC = G == 1 && P * K <= 9 ? 2 : 1;                 // column halves whose activations are held at once
    extern __shared__ __attribute__((aligned(16))) float part[];     // [wavefront][row tile][token][row]
    const int tid = threadIdx.x, lane = tid & 63, nw = (int)blockDim.x >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, q = lane >> 4;
    int o = 0;
    while (o + 1 < args.nops && (int)blockIdx.x >= args.op[o + 1].wg0) ++o;
    const Op &op = args.op[o];
    const int out = op.out, in = op.in, T = args.T;
    const int RT = row_tiles(out), CT = col_tiles(in);
    const int rt0 = ((int)blockIdx.x - op.wg0) * P;

    // the row tiles of this workgroup; one past the end of the matrix reads the last one (not stored)
    const uint32_t *bits[P];
#pragma unroll
    for (int p = 0; p < P; ++p) bits[p] = op.bits + (size_t)min(rt0 + p, RT - 1) * CT * tile_words(K) + lane * 2 * K;

    Words<K> w[P];
    if (wave < CT)
#pragma unroll
        for (int p = 0; p < P; ++p) w[p] = load_words<K>(bits[p] + (size_t)wave * tile_words(K));
    v4f acc[P][K][G];
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int g = 0; g < G; ++g) acc[p][k][g] = (v4f){0.f, 0.f, 0.f, 0.f};

    // columns of this lane: 32 consecutive ones per half of a column tile, all of them inside the
    // matrix or none (in % 32 == 0); lane r of a row of 16 feeds token r
    const uint16_t *xrow[G];
#pragma unroll
    for (int g = 0; g < G; ++g)
        xrow[g] = static_cast<const uint16_t *>(op.x) + (size_t)min(16 * g + r, T - 1) * in + 32 * q;

    for (int ct = wave; ct < CT; ct += nw) {
        const int j0 = ct * TILE_COLS;
        // scales: lane r of a row of 16 holds the pair of columns 2 r, 2 r + 1 of the row's 32
        uint32_t hw[2][K];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const bool real = j0 + 128 * c + 32 * q < in;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const uint16_t *hp = op.h + (size_t)k * in + (real ? j0 + 128 * c + 32 * q + 2 * r : 0);
                uint32_t v;
                if (op.h_even) v = *reinterpret_cast<const uint32_t *>(hp);
                else v = (uint32_t)hp[0] | ((uint32_t)hp[1] << 16);      // the scales need only be 2-byte aligned
                hw[c][k] = real ? v : 0u;
            }
        }
        uint4 x[XC][4][G];
        auto load_x = [&](int c) {
            const bool real = j0 + 128 * c + 32 * q < in;
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    x[c % XC][s][g] = make_uint4(0u, 0u, 0u, 0u);
                    if (real) x[c % XC][s][g] = *reinterpret_cast<const uint4 *>(xrow[g] + j0 + 128 * c + 8 * s);
                }
        };
        load_x(0);
        if constexpr (XC == 2) load_x(1);
        Words<K> next[P];
        if (AHEAD && ct + nw < CT)
#pragma unroll
            for (int p = 0; p < P; ++p) next[p] = load_words<K>(bits[p] + (size_t)(ct + nw) * tile_words(K));
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            if (XC == 1 && c == 1) load_x(1);
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                v8h b[G];
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    uint4 v = x[c % XC][s][g];
                    if constexpr (BF16) v = make_uint4(half_of_bf16_pair(v.x), half_of_bf16_pair(v.y), half_of_bf16_pair(v.z), half_of_bf16_pair(v.w));
                    b[g] = __builtin_bit_cast(v8h, v);
                }
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    uint32_t hp[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) hp[j] = row_lane(hw[c][k], 4 * s + j);
#pragma unroll
                    for (int p = 0; p < P; ++p) {
                        // element e of the lane's eight is column 8 s + e: native bit 4 e + s.  Shifted by
                        // 7 - s (3 - s) bit 8 j + s (8 j + 4 + s), of element 2 j (2 j + 1), is the
                        // top of byte j; a permute brings the two bytes to the tops of the halves
                        const uint32_t even = w[p].w[c * K + k] << (7 - s), odd = w[p].w[c * K + k] << (3 - s);
                        uint4 a;
                        uint32_t *const av = reinterpret_cast<uint32_t *>(&a);
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            av[j] = hp[j] ^ (__builtin_amdgcn_perm(odd, even, (uint32_t)((4 + j) << 24 | j << 8)) & 0x80008000u);
                        const v8h av8 = __builtin_bit_cast(v8h, a);
#pragma unroll
                        for (int g = 0; g < G; ++g) acc[p][k][g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(av8, b[g], acc[p][k][g], 0, 0, 0);
                    }
                }
            }
        }
        if (AHEAD) {
#pragma unroll
            for (int p = 0; p < P; ++p) w[p] = next[p];
        } else if (ct + nw < CT) {
#pragma unroll
            for (int p = 0; p < P; ++p) w[p] = load_words<K>(bits[p] + (size_t)(ct + nw) * tile_words(K));
        }
    }

    // ---- partial outputs of this wavefront: path sum with the output scales (Section 4.1).  Lane
    // (r, q) holds token r, rows 4 q .. 4 q + 3 of the row tile.
#pragma unroll
    for (int p = 0; p < P; ++p) {
        float gq[K][4];
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = min((rt0 + p) * TILE_ROWS + 4 * q + i, out - 1);
                gq[k][i] = __half2float(__ushort_as_half(op.g[(size_t)k * out + row])) * (BF16 ? 2.f : 1.f);
            }
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
    constexpr int lds_max = max_waves(G) * P * G * 1024;
    if (lds_max > 64 * 1024) {
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
    hipLaunchKernelGGL((batch_kernel<K, G, P, BF16>), dim3((unsigned)groups), dim3((unsigned)(nw * 64)), nw * P * G * 1024, stream, args);
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
        args.op[i].h_even = ((uintptr_t)args.op[i].h & 3) == 0;
    }
    Shape s;
    s.K = K;
    const int G = token_groups(args.T);
    s.P = row_tiles_per_wg(RT, args.nops, K, G);
    s.groups = 0;
    for (int i = 0; i < args.nops; ++i) {
        args.op[i].wg0 = s.groups;
        s.groups += (RT[i] + s.P - 1) / s.P;
    }
    s.nw = std::min(CT, max_waves(G));      // a wavefront takes whole column tiles
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
    o.wg0 = 0; o.h_even = 0;
    return o;
}

bool call_supported(const rb_layer *L, int T) { return (L->K == 2 || L->K == 3) && T >= 1 && T <= CALL_MAX_T && L->in % 32 == 0; }

int launch_call(const rb_layer *L, const void *X, void *Y, int T, int act_dtype, int out_dtype, hipStream_t stream)
{
    Args args;
    args.nops = 1; args.T = T; args.out_dtype = out_dtype;
    args.op[0] = make_op(*L, X, Y);
    const Shape s = shape_of(args, L->K);
    const int rc = act_dtype == RB_BF16 ? launch_shape<true>(args, s, stream) : launch_shape<false>(args, s, stream);
    if (rc != RB_OK) return rc;
    return hipGetLastError() == hipSuccess ? RB_OK : RB_ERR_HIP;
}

bool layer_supported(const rb_layer *L, int T)
{
    return (L->K == 2 || L->K == 3) && T >= 1 && T <= STACK_MAX_T && L->in % 32 == 0;
}

// A plan lives on the host: the kernel needs nothing in device memory besides the buffers.  The
// workspace is the name it is run by.
size_t plan_workspace_bytes() { return 256; }

struct Prepared { std::vector<std::pair<Args, Shape>> launches; };
static std::mutex g_mutex;
static std::map<const void *, std::shared_ptr<const Prepared>> g_prepared;

int prepare_plan(const rb_layer *layers, const rb_stack_op *sops, int n_ops, uint16_t *const *bufs, int T,
                 void *workspace, size_t workspace_bytes_)
{
    if (T < 1 || T > STACK_MAX_T) return RB_ERR_UNSUPPORTED;
    if (!workspace || workspace_bytes_ < plan_workspace_bytes()) return RB_ERR_WORKSPACE;
    // an op that reads another one's output reads all of it
    std::map<int, int> width;
    for (int n = 0; n < n_ops; ++n) {
        const rb_layer &L = layers[sops[n].layer];
        if (!layer_supported(&L, T)) return RB_ERR_UNSUPPORTED;
        const auto it = width.find(sops[n].src);
        if (it != width.end() && it->second != L.in) return RB_ERR_SHAPE;
        width[sops[n].dst] = L.out;
    }
    // launches: runs of consecutive ops of one K that neither read nor overwrite each other
    auto pr = std::make_shared<Prepared>();
    for (int op0 = 0; op0 < n_ops;) {
        Args args;
        args.nops = 0; args.T = T; args.out_dtype = RB_F16;
        const int K = layers[sops[op0].layer].K;
        for (int n = op0; n < n_ops && args.nops < MAX_STAGE_OPS; ++n) {
            const rb_layer &L = layers[sops[n].layer];
            bool conflict = L.K != K;
            for (int m = op0; m < n; ++m)
                if (sops[m].dst == sops[n].src || sops[m].dst == sops[n].dst || sops[m].src == sops[n].dst) conflict = true;
            if (conflict) break;
            args.op[args.nops++] = make_op(L, bufs[sops[n].src], bufs[sops[n].dst]);
        }
        const Shape s = shape_of(args, K);
        pr->launches.emplace_back(args, s);
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
    if (workspace_bytes_ < plan_workspace_bytes()) return RB_ERR_WORKSPACE;
    for (const auto &l : pr->launches) {
        const int rc = launch_shape<false>(l.first, l.second, stream);
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
