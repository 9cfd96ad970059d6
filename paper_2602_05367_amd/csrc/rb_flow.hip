// Three and four tokens of two-path layers whose ops have much to do (takes_flow in rb_plan.h; the others keep the step lists of rb_mx.hip): set-up
// kernels, the persistent kernel, and its host planner.  See rb_flow.h for the layout of the operands and rb_mx.h for the arithmetic.
//
// The persistent kernel runs one workgroup per compute unit through the stages of the plan:
//   * the row tiles of a stage's ops, one op after the other, are dealt to the workgroups in contiguous shares, so that a
//     workgroup nearly always works on one op; each of eight wavefronts takes a run of column tiles of all the share's row
//     tiles: it fetches the operands of its columns once and multiplies them with one pair of row tiles after the other;
//   * a ninth wavefront streams the shares' sign tiles, one after the other, into a ring in LDS, across stages, as far as there is room.
//     Asked for by the wavefronts that use them, they took 8.5 us a stage: about 20 KB can be on their way to a compute unit, and a
//     wavefront that asks for more stands still;
//   * partial sums of the wavefronts meet in LDS; then every wavefront finishes rows (where there are fewer row tiles than
//     wavefronts, several share one): y = sum_k g_k * acc_k, fp16 rounding, and the four-term expansion of h (.) y for the ops that read y
//     next, written with device-scope 16-byte stores, before y itself;
//   * hand-over between compute units: before a launch every 16-byte group of an expanded input
//     that a producer of the launch will write is filled with 0xff bytes, which no bf8 term of a
//     finite value has.  Producers just store.  A wavefront waits a fixed pause after its workgroup's sums, requests its
//     operand tiles with plain loads (shared by the 32 compute units of an XCD in its L2)
//     and checks every 32-bit word of them; only tiles with a
//     word that still reads 0xffffffff are waited for and read again past the L2.  The pause is a
//     matter of speed, not of correctness.
//
// What bounds it: latencies and instruction issue.  A stage of the 7B-shaped chain takes 7.1 us at three and four tokens, one of its decoder blocks 7.9: by time
// stamps of all wavefronts, on the mean, the pause 1.5 and 1.4, operands 1.5 and 2.2 (5 and 3 % of the tiles late), products 1.9 and 1.6 (two matrix
// instructions and 16 vector instructions per 1 KB of signs and path, 25 per row tile for the sums over terms), sums of squares and what is added 0 and 0.4, until the
// slowest wavefront has filed its sums 1.0 and 1.3, finishing rows 0.4 and 0.6, tables 0.7 and 0.6.
// Measured, 7B-shaped, in dependency order (before: the step-list kernel): three tokens 1235 -> 920 us, decoder blocks at three 1306 -> 1020; 13B-shaped at four, 16
// blocks 969 -> 687, with norms and residuals 1037 -> 795; 16 blocks of 2048 x 5504 at three 397 -> 318.  Fewer tokens stay on the step-list kernel: this form
// takes 770 us at one (641 there), at two 795 (839), but 930 for decoder blocks (852) and 355 for 16 blocks of 2048 columns (253).
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>

#include <atomic>
#include <cmath>
#include <cstring>
#include <map>
#include <memory>
#include <mutex>
#include <type_traits>
#include <vector>

#include "rabit.h"
#include "rb_internal.h"
#include "rb_layout.h"
#include "rb_flow.h"
#include "rb_mx_device.h"
#include "rb_plan.h"

namespace rb {
namespace flow {

using namespace rb::mx;

// Pointers read from the op table are generic; dereferencing them as such makes FLAT instructions,
// which also count as LDS traffic: every LDS wait would then wait for global stores to be acknowledged.
#define RB_GLOBAL(T, p) ((__attribute__((address_space(1))) T *)(p))

// Hand-over timing (a matter of speed only: a consuming wavefront checks what it gets), in units of 64 clocks, 27 ns: between a wavefront's own stores of a
// stage and its first request of the next one's operands.  (us without it, with 24, 32, 40, 48, 64 units: 7B-shaped chain at three tokens
// 1007 924 913 904 899 928, decoder blocks at three 1025 1012 1005 991 981 1019, of 13B at four, 16 of them, 802 803 801 800 794 775, 2048-wide chain at three
// 335 318 316 316 321 343)
constexpr int GO_PAUSE = 48;
// between two looks at a tile that was not yet written (units of 64 clocks): the first 64 come quickly, the rest far
// apart (wavefronts that look too often keep the stores they wait for from landing)
constexpr uint32_t MAX_LOOKS = 0x40000, QUICK_LOOKS = 64;

// ------------------------------------------------------------ prep kernel ---
// One workgroup per op: power-of-two scale of each path's input scales and the zero fill of the
// expanded-input array (padding columns and unused operand columns must read as zero).
__global__ __launch_bounds__(256) void prep_kernel(Op *ops, uint32_t *error)
{
    const int o = blockIdx.x;
    Op &op = ops[o];
    __shared__ float red[256];
    for (int p = 0; p < K; ++p) {
        float m = 0.f;
        for (int j = threadIdx.x; j < op.in; j += 256)
            m = fmaxf(m, fabsf(__half2float(reinterpret_cast<const __half *>(op.h)[(size_t)p * op.in + j]) * norm_weight(op, j)));
        red[threadIdx.x] = m;
        __syncthreads();
        for (int s = 128; s > 0; s >>= 1) {
            if ((int)threadIdx.x < s) red[threadIdx.x] = fmaxf(red[threadIdx.x], red[threadIdx.x + s]);
            __syncthreads();
        }
        if (threadIdx.x == 0) {
            const float sc = input_scale(red[0]);
            op.sc[p] = sc;
            op.inv_sc[p] = 1.f / sc;
        }
        __syncthreads();
    }
    const size_t n16 = up_bytes(op.in) / 16;
    uint4 *up = reinterpret_cast<uint4 *>(op.up);
    for (size_t i = threadIdx.x; i < n16; i += 256) up[i] = make_uint4(0, 0, 0, 0);
    if (o == 0 && threadIdx.x < 2) error[threadIdx.x] = 0;      // the give-up mark and the count of tiles waited for
}

// Second set-up pass (needs the scales of every op): the tables of the flow kernel.  One workgroup per (stage, LINK_GROUPS
// workgroups of the flow kernel), half of it per workgroup; a thread per (slot, row).
constexpr int LINK_GROUPS = 8;
__global__ __launch_bounds__(256) void link_kernel(const Op *ops, const Stage *stages, int G, Work *work, SlotRec *slots, float *vals,
                                                   SlotExt *ext, const uint8_t *up0)
{
    const int st = blockIdx.x;
    const Stage &stage = stages[st];
    // the op and row tile at place t of the stage's row tiles
    auto find = [&](uint32_t t, uint32_t &rt) {
        int i = 0;
        for (; i + 1 < stage.nops && t >= (uint32_t)stage.rt[i]; ++i) t -= (uint32_t)stage.rt[i];
        rt = t;
        return stage.op0 + i;
    };
    const int slot = (threadIdx.x >> 4) & 7, row = threadIdx.x & 15;
    for (int sub = 0; sub < LINK_GROUPS / 2; ++sub) {
        const int grp = (int)blockIdx.y * LINK_GROUPS + 2 * sub + (int)(threadIdx.x >> 7);
        if (grp >= G) continue;
        uint32_t t0, t1;
        share_of((uint32_t)stage.tiles, (uint32_t)grp, (uint32_t)G, t0, t1);
        const uint32_t rec = stage.rec0 + (uint32_t)grp * (uint32_t)stage.n_slots;
        if ((threadIdx.x & 127) == 0) {
            Work w = {};
            int seg = 0;
            uint32_t c = 0;
            for (int i = 0; i < stage.nops; ++i) {
                const Op &op = ops[stage.op0 + i];
                const uint32_t c0 = stage.gated ? 0u : c, e = c0 + (uint32_t)stage.rt[i];
                const uint32_t a = t0 > c0 ? t0 : c0, b = t1 < e ? t1 : e;
                c = e;
                if (a >= b) continue;
                if (seg < 2) {
                    w.bits[seg] = (uint64_t)op.bits + (uint64_t)(a - c0) * (uint32_t)(op.CT * 512 * K);
                    w.up[seg] = (uint32_t)((op.up - up0) / 256);
                    w.P[seg] = (uint16_t)(b - a);
                    w.CT[seg] = (uint16_t)op.CT;
                    if (seg == 1) w.slot1 = (uint8_t)(stage.gated ? GATED_SLOTS : a - t0);
                    if (op.dep >= 0) w.flags |= (uint8_t)(WORK_DEP0 << seg);
                }
                ++seg;
            }
            if (seg < 1) w.CT[0] = 1;
            if (seg < 2) w.CT[1] = 1;
            const Op &op = ops[stage.op0];
            w.n_fin = (uint8_t)(t1 - t0);
            if (stage.gated) w.flags |= WORK_GATED;
            w.rec = rec;
            if (stage.norm) {
                w.flags |= WORK_NORM;
                w.ssq_in = (uint32_t)((reinterpret_cast<const uint8_t *>(op.ssq_in) - up0) / 256);
                w.n_part = (uint32_t)op.n_part;
                w.inv_n = 1.f / (float)op.in;
            }
            work[(size_t)st * G + grp] = w;
        }
        if (slot >= stage.n_slots) continue;
        // (of a gate-times-up stage the slots from GATED_SLOTS on hold the up projection's output scales)
        uint32_t rt = 0;
        int my_op = -1;
        if (stage.gated) {
            if (t0 + (uint32_t)(slot % GATED_SLOTS) < t1) { my_op = stage.op0 + slot / GATED_SLOTS; rt = t0 + (uint32_t)(slot % GATED_SLOTS); }
        } else if (t0 + (uint32_t)slot < t1) {
            my_op = find(t0 + (uint32_t)slot, rt);
        }
        SlotRec sr = {};
        SlotExt sx = {};
        float v[VALS_ROW];
        for (float &x : v) x = 0.f;
        if (my_op >= 0) {
            const Op &op = ops[my_op];
            const int row0 = (int)rt * 16, grow = row0 + row;
            const bool valid = grow < op.out;
            sr.y = op.y ? (uint64_t)(op.y + row0) : 0;
            sr.out = op.out; sr.n_cons = (uint8_t)op.n_cons; sr.rows = (uint8_t)min(16, op.out - row0); sr.resid_kind = (uint8_t)op.resid_kind;
            if (op.resid_kind != RESID_NONE) sx.resid = (uint64_t)op.resid + (uint64_t)row0 * (op.resid_kind == RESID_COPY ? 4u : 2u);
            if (op.ssq_out) sx.ssq_out = (uint32_t)((reinterpret_cast<const uint8_t *>(op.ssq_out) - up0) / 4 + rt);
            sx.ssq_stride = op.RT;
            if (op.rcopy) sx.rcopy = (uint32_t)((reinterpret_cast<const uint8_t *>(op.rcopy) - up0) / 4 + row0);
            for (int k = 0; k < K && valid; ++k) v[k] = __half2float(reinterpret_cast<const __half *>(op.g)[(size_t)k * op.out + grow]) * op.inv_sc[k];
            for (int c = 0; c < op.n_cons; ++c) {
                const Op &m = ops[op.cons[c]];
                sr.up[c] = (uint32_t)((m.up + up_group_offset(row0, 0, 0) - up0) / 16);
                const float w = valid ? norm_weight(m, grow) : 0.f;
                for (int k = 0; k < K && valid; ++k) v[K + c * K + k] = __half2float(reinterpret_cast<const __half *>(m.h)[(size_t)k * m.in + grow]) * w * m.sc[k];
            }
        }
        const size_t idx = rec + (size_t)slot;
        for (int i = 0; i < VALS_ROW; ++i) vals[(idx * 16 + (size_t)row) * VALS_ROW + i] = v[i];
        if (row == 0) {
            slots[idx] = sr;
            if (ext) ext[idx] = sx;
        }
    }
}

// --------------------------------------------------------- expand kernel ---
// Input scaling u_k = h_k (.) x (Section 4.1) for ops whose input comes from
// outside the fused ops, written as four bf8 terms in operand order.  A thread takes 16 consecutive
// columns of one token and path (in % 32 == 0) and stores one 16-byte group per term.
__device__ __forceinline__ void expand_part(const Op *ops, const int *which, int bx, int tok, int bz)
{
    const Op &op = ops[which[bz]];
    const int nblk = op.in / 16;
    const int id = bx * 256 + (int)threadIdx.x;
    if (id >= nblk * K) return;
    const int p = id / nblk, j0 = (id - p * nblk) * 16;
    const uint4 *xs = reinterpret_cast<const uint4 *>(op.x + (size_t)tok * op.in + j0);     // buffers are 16-byte aligned
    const uint4 xq[2] = {xs[0], xs[1]};
    const uint32_t xw[8] = {xq[0].x, xq[0].y, xq[0].z, xq[0].w, xq[1].x, xq[1].y, xq[1].z, xq[1].w};
    const __half *hp = reinterpret_cast<const __half *>(op.h) + (size_t)p * op.in + j0;     // scales: 2-byte aligned
    uint32_t out[4][4] = {};                                  // [term][word of the group]
    const float sc = op.sc[p];
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        const float x = __half2float(__ushort_as_half((unsigned short)(xw[e >> 1] >> (16 * (e & 1)))));
        const uint32_t terms = expand4(__half2float(hp[e]) * norm_weight(op, j0 + e) * x * sc);
#pragma unroll
        for (int t = 0; t < 4; ++t) out[t][e >> 2] |= ((terms >> (8 * t)) & 0xffu) << (8 * (e & 3));
    }
#pragma unroll
    for (int t = 0; t < 4; ++t)
        *reinterpret_cast<uint4 *>(op.up + up_group_offset(j0, p, 4 * tok + t)) =
            make_uint4(out[t][0], out[t][1], out[t][2], out[t][3]);
}

// Before every launch: the expanded input of every op that a producer of this
// launch will write is set to "not written yet" (0xff in every byte of the 16-byte groups of real
// columns: no bf8 term of a finite value is 0xff; padding columns read as zero).  POISON_SPLIT
// workgroups per op.
constexpr int POISON_SPLIT = 4;
__device__ __forceinline__ void poison_part(const Op *ops, int n_ops, uint4 *aux, size_t aux16, int bx, int by)
{
    if (bx == n_ops) {
        // what finishing wavefronts hand to each other in a decoder block: no sum of squares and
        // no fp16 value in a word of its own is all ones
        for (size_t i = by * 256 + threadIdx.x; i < aux16; i += 256 * POISON_SPLIT)
            aux[i] = make_uint4(0xffffffffu, 0xffffffffu, 0xffffffffu, 0xffffffffu);
        return;
    }
    const Op &op = ops[bx];
    if (op.dep < 0) return;
    const int per16 = K * 4 * T, groups = (int)(up_bytes(op.in) / 16);
    uint4 *up = reinterpret_cast<uint4 *>(op.up);
    for (int i = by * 256 + (int)threadIdx.x; i < groups; i += 256 * POISON_SPLIT) {
        // which 16 input columns group i holds: [128-column block][half][q]
        const int c = i / per16;
        const uint32_t v = (c >> 3) * 128 + (c >> 2 & 1) * 64 + (c & 3) * 16 < op.in ? 0xffffffffu : 0u;
        up[i] = make_uint4(v, v, v, v);
    }
}

// What goes before the flow kernel in every run, as one launch: the first n_poison workgroups mark
// inputs (they write the expanded inputs of ops fed from inside the launch), the next n_expand
// expand the inputs from outside (ex x ey x ez workgroups; they write those of the other ops), and
// in a decoder block the next n_ssq add up the squares of the inputs from outside that an op normalises
// (one workgroup per such input and token) and the rest put aside what ops add of the caller's.
__global__ __launch_bounds__(256) void before_kernel(const Op *ops, int n_ops, const int *which, int n_poison,
                                                     int n_expand, int ex, int ey, int n_ssq, uint4 *aux, size_t aux16)
{
    const int b = (int)blockIdx.x;
    if (b < n_poison) {
        poison_part(ops, n_ops, aux, aux16, b / POISON_SPLIT, b % POISON_SPLIT);
        return;
    }
    const int e = b - n_poison;
    if (e < n_expand) {
        expand_part(ops, which, e % ex, (e / ex) % ey, e / (ex * ey));
        return;
    }
    const int q = e - n_expand;
    if (q < n_ssq) {
        ssq_part(ops, which, q / ey, q % ey);
        return;
    }
    aside_part(ops, ey, (q - n_ssq) / ASIDE_SPLIT, (q - n_ssq) % ASIDE_SPLIT);
}

// ---------------------------------------------------------- flow kernel ---
// a store that passes the L2 of this XCD (for another XCD's wavefront to read with a device-scope load)
__device__ __forceinline__ void store_sc1_u32(uint64_t addr, uint32_t v)
{
    asm volatile("global_store_dword %0, %1, off sc1" : : "v"(addr), "v"(v) : "memory");
}
// what a wavefront that gave up a bounded wait leaves in the plan's error word (rb_stack_status
// reports any of them as RB_ERR_HANDOVER; rb_stack_gave_up tells which)
constexpr int GAVE_UP_TILE = 1;       // an input tile was never written
constexpr int GAVE_UP_TORN = 2;       // a tile whose first bytes had arrived kept reading as unwritten
constexpr int GAVE_UP_GO = 3;         // a sign tile was never announced inside the workgroup
constexpr int GAVE_UP_BLOCK = 4;      // a sum of squares or a residual value of a decoder block never arrived

#define RB_LDS(p) ((__attribute__((address_space(3))) void *)(p))
constexpr int LOAD_SC1 = 16, LOAD_NT = 2;                // cache policies of loads
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer(const void *p, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00020000);
}

// the operand of a column tile: [128-column block][path][half of the contraction]
struct Tile { v4i half[2][K][2]; };

// Row tiles that a workgroup's share has of one op
struct Segment {
    uint64_t bits;            // sign tiles of the first row tile
    uint32_t up;              // expanded input, see Work
    int P, CT;                // row tiles (0: there is no such segment), column tiles
    int slot0;                // where the sums of the first row tile go
    bool dep;                 // the input is written inside the launch
};
// LDS: partial sums [stage parity][slot][wavefront][path][token][row], root mean squares [stage parity][token], counters, then the
// sign tiles, a ring that the loading wavefront fills in the order of the workgroup's shares
struct Lds {
    static constexpr int PART = K * T * 16;                               // floats of a wavefront and row tile
    static constexpr int RINV_OFF = 2 * MAXSLOT * CWAVES * PART * 4;
    static constexpr int USED_OFF = RINV_OFF + 32;                        // per wavefront: the first tile of the stream that it still needs
    static constexpr int LANDED_OFF = USED_OFF + 4 * CWAVES;              // tiles of the stream that have arrived
    static constexpr int ARRIVED_OFF = LANDED_OFF + 4;                       // wavefronts that have filed their sums, over all stages
    static constexpr int SIGNS_OFF = RINV_OFF + 128;
    static constexpr int TILE_BYTES = 512 * K;
    static constexpr int TILES = (160 * 1024 - SIGNS_OFF) / TILE_BYTES;
    static constexpr int BYTES = SIGNS_OFF + TILES * TILE_BYTES;
    static_assert(ARRIVED_OFF + 4 <= SIGNS_OFF, "counters");
};
__device__ __forceinline__ uint32_t lds_read(uint32_t at)
{
    uint32_t v;
    asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(v) : "v"(at) : "memory");
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}
__device__ __forceinline__ void lds_write(uint32_t at, uint32_t v) { asm volatile("ds_write_b32 %0, %1" : : "v"(at), "v"(v) : "memory"); }
__device__ __forceinline__ void lds_add(uint32_t at, uint32_t v) { asm volatile("ds_add_u32 %0, %1" : : "v"(at), "v"(v) : "memory"); }

// What a producer stores carries its own validity (a 16-byte group of an expanded input is all 0xff
// until it is written), so a producer neither waits for its stores to be acknowledged nor raises a
// flag, and nobody polls memory for flags.
// BLK: the form that runs decoder blocks (normalised inputs, gate times up, residual additions when rows are finished).  LEFT_OUT: a stage has fewer row
// tiles than there are workgroups.  (Of two forms: with the longer pause in it the other one of decoder blocks takes 1 % longer)
template <bool BLK, bool LEFT_OUT>
__global__ __launch_bounds__(THREADS, 3) void flow_kernel(const Work *__restrict__ work,
                                                           const SlotRec *__restrict__ slots, const float *__restrict__ vals,
                                                           const SlotExt *__restrict__ ext, uint8_t *up0, uint32_t *__restrict__ error,
                                                           int n_stages, int tokens, int go_pause, float eps)
{
    constexpr int C = 4 * T;                                 // operand columns of a path
    constexpr int TILE_BYTES = Lds::TILE_BYTES, PART = Lds::PART, TILES = Lds::TILES;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t grp = blockIdx.x, n_groups = gridDim.x;
    const int col = lane & 15, qd = lane >> 4;
    const int scale_b = term_scale(col);
    const uint32_t opnd_lane = (uint32_t)(qd * K * C + col) * 16u;
    uint32_t c22;
    asm volatile("v_mov_b32 %0, 0x22222222" : "=v"(c22));
    auto lds_at = [&](int offset) -> uint32_t { return (uint32_t)(size_t)RB_LDS(lds) + (uint32_t)offset; };
    uint32_t waited = 0;                                     // tiles found not yet written
    bool failed = false;                                     // a producer never delivered: stop waiting, report
    auto give_up = [&](int reason) {
        failed = true;
        if (lane == 0) __hip_atomic_store(RB_GLOBAL(uint32_t, error), (uint32_t)reason, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };

    auto first_of = [&](const Work &w) { return Segment{w.bits[0], w.up[0], w.P[0], w.CT[0], 0, (w.flags & WORK_DEP0) != 0}; };
    auto second_of = [&](const Work &w) { return Segment{w.bits[1], w.up[1], w.P[1], w.CT[1], w.slot1, (w.flags & WORK_DEP1) != 0}; };
    uint8_t *const signs = lds + Lds::SIGNS_OFF;
    auto columns_of = [&](const Segment &s) { return run_begin(wave + 1, s.CT) - run_begin(wave, s.CT); };
    // LDS set-up.  (The compiler does not count stores made in assembly: it need not wait for them at the barrier, and a zero that came
    // late could undo an arrival, for which the others would wait without an end)
    if (threadIdx.x < 16) lds_write(lds_at(Lds::USED_OFF) + threadIdx.x * 4, 0u);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __syncthreads();

    if (wave == CWAVES) {
        // ======================= loading wavefront ==========================
        // A workgroup's share of an op is one contiguous run of tiles
        constexpr uint32_t FLIGHT = 12;                       // tiles on their way when it looks around (8 to 24: the same)
        __builtin_amdgcn_s_setprio(3);
        uint32_t issued = 0, used = 0, told = 0;              // tiles asked for, given back, announced
        int slot = 0;
        Work w = work[grp];
#pragma unroll 1
        for (int st = 0; st < n_stages; ++st) {
            const Work next = work[(size_t)min(st + 1, n_stages - 1) * n_groups + grp];
#pragma unroll 1
            for (int n = 0; n < 2; ++n) {
                const Segment s = n == 0 ? first_of(w) : second_of(w);
                const int count = s.P * s.CT;
                const uint8_t *tile = reinterpret_cast<const uint8_t *>(s.bits) + lane * 16;
                if (s.P == 0) break;
                // (four tiles at a time: what is done for each of them bounds the rate)
#pragma unroll 1
                for (int j = 0; j < count;) {
                    const int m = min(min(4, count - j), TILES - slot);
                    asm volatile("s_waitcnt vmcnt(%0)" : : "n"(FLIGHT) : "memory");
                    if (issued - told > FLIGHT) {
                        told = issued - FLIGHT;
                        if (lane == 0) lds_write(lds_at(Lds::LANDED_OFF), told);
                    }
                    if (!ring_has_room(issued, (uint32_t)m, used, TILES)) {
                        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                        told = issued;
                        if (lane == 0) lds_write(lds_at(Lds::LANDED_OFF), told);
                        for (;;) {
                            uint32_t u;
                            asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(u) : "v"(lds_at(Lds::USED_OFF) + (lane & (CWAVES - 1)) * 4) : "memory");
                            u -= issued;                      // (the least of eight, as numbers that may wrap)
#pragma unroll
                            for (int i = 1; i < CWAVES; i <<= 1) u = (uint32_t)min((int)u, __shfl_xor((int)u, i));
                            used = issued + (uint32_t)__builtin_amdgcn_readfirstlane((int)u);
                            if (ring_has_room(issued, (uint32_t)m, used, TILES)) break;
                            __builtin_amdgcn_s_sleep(1);
                        }
                    }
                    uint8_t *const at = signs + slot * TILE_BYTES;
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (i < m) {
                            // non-temporal: every sign tile is read once
                            __builtin_amdgcn_global_load_lds(tile + i * TILE_BYTES, RB_LDS(at + i * TILE_BYTES), 16, 0, LOAD_NT);
                        }
                    tile += m * TILE_BYTES;
                    slot = slot + m == TILES ? 0 : slot + m;
                    issued += (uint32_t)m;
                    j += m;
                }
            }
            w = next;
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (lane == 0) lds_write(lds_at(Lds::LANDED_OFF), issued);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        return;
    }

    // ======================= computing and finishing ==========================
    uint32_t landed = 0;
    auto wait_landed = [&](uint32_t count) {
        for (uint32_t spins = 0; (int)(landed - count) < 0 && !failed; ++spins) {
            landed = lds_read(lds_at(Lds::LANDED_OFF));
            if ((int)(landed - count) >= 0) break;
            __builtin_amdgcn_s_sleep(1);
            if (spins > (1u << 24)) give_up(GAVE_UP_GO);
        }
    };
    auto still_needs = [&](uint32_t tile) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");    // what comes before it has been read
        if (lane == 0) lds_write(lds_at(Lds::USED_OFF) + wave * 4, tile);
    };
    auto load_operand = [&](Tile &t, uint32_t up, int ct, auto policy) {
        const auto rs = buffer(up0 + (uint64_t)up * 256 + (uint64_t)ct * (2 * UP_BLOCK_BYTES), 2 * UP_BLOCK_BYTES);
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int k = 0; k < K; ++k)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    t.half[c][k][j] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)opnd_lane + k * (C * 16), (c * 2 + j) * (4 * K * C * 16), decltype(policy)::value));
    };
    // a word of the tile that has not been written
    auto unwritten = [&](const Tile &t) -> bool {
        uint32_t half[2] = {0, 0};                            // (two chains)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int k = 0; k < K; ++k)
#pragma unroll
                for (int e = 0; e < 8; ++e) half[c] = max(half[c], (uint32_t)t.half[c][k][e >> 2][e & 3]);
        const uint32_t all = max(half[0], half[1]);
        return all == 0xffffffffu;
    };
    // A 32-bit word that reads 0xffffffff has not been written (its producer was late, the L2 of this XCD got hold of the line
    // before it was written, or a 16-byte store has landed in part): the first words of all groups of the tile are looked at past
    // the L2 until they are there
    auto look = [&](uint32_t up, int ct) {
        const auto rs = buffer(up0 + (uint64_t)up * 256 + (uint64_t)ct * (2 * UP_BLOCK_BYTES), 2 * UP_BLOCK_BYTES);
        uint32_t looks = 0;
        bool missing;
        do {
            uint32_t most = 0;
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int k = 0; k < K; ++k)
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const uint32_t v = __builtin_amdgcn_raw_buffer_load_b32(rs, (int)opnd_lane + k * (C * 16), (c * 2 + j) * (4 * K * C * 16), LOAD_SC1);
                        most = max(most, v & 0xffu);
                    }
            missing = __ballot(most == 0xffu) != 0ull;
            if (missing) {
                __builtin_amdgcn_s_sleep(8);
                if (looks > QUICK_LOOKS) __builtin_amdgcn_s_sleep(56);
                ++looks;
            }
            asm volatile("" ::: "memory");                   // (every look is a load of its own)
        } while (missing && looks < MAX_LOOKS);
        if (missing) give_up(GAVE_UP_TILE);
    };

    // ---- a segment: the wavefront's column tiles of all its row tiles, two row tiles at a time.  The operands of up to M column tiles are held in
    // registers; of a longer run they are fetched anew for every row tile.  `base` is the number of the segment's first tile in the stream, at
    // `ring` in LDS.
    auto multiply = [&](auto m_const, const Segment &s, uint32_t base, int ring, int parity) {
        constexpr int M = decltype(m_const)::value;
        const int c0 = run_begin(wave, s.CT), n = columns_of(s);
        // the first tile that this wavefront needs from row tile p on (what comes after the segment may be cut into other runs)
        auto row_of = [&](int p) { return base + (uint32_t)(p * s.CT + (p < s.P ? c0 : 0)); };
        Tile b[M];
        auto request = [&](int piece, int m) {
            auto ask = [&](auto policy) {
#pragma unroll
                for (int d = 0; d < M; ++d)
                    if (d < m) load_operand(b[d], s.up, c0 + piece + d, policy);
            };
            auto missing = [&]() -> bool {
                bool any = false;
#pragma unroll
                for (int d = 0; d < M; ++d)
                    if (d < m) any |= unwritten(b[d]);
                return __ballot(any) != 0ull;
            };
            ask(std::integral_constant<int, 0>());
            bool late = missing() && s.dep;
            int again = 0;
            if (late)
#pragma unroll
                for (int d = 0; d < M; ++d)
                    if (d < m && __ballot(unwritten(b[d])) != 0ull) ++waited;
            while (late && !failed && again < 6) {
                asm volatile("" ::: "memory");
#pragma unroll 1
                for (int d = 0; d < m; ++d) look(s.up, c0 + piece + d);
                ask(std::integral_constant<int, LOAD_SC1>());
                ++again;
                late = missing();
            }
            // a group whose store had landed in part is complete one look later; a word that stays unwritten is
            // reported, not trusted
            if (late && !failed) give_up(GAVE_UP_TORN);
        };
        struct Words { uint32_t w[2 * K]; };
        auto wrapped = [&](int at) {
            while (at >= TILES) at -= TILES;
            return at;
        };
        // (at: a place in the ring, or less than M beyond its end)
        auto read_tile = [&](int at) -> Words {
            Words r;
            const uint8_t *const tile = signs + (at >= TILES ? at - TILES : at) * TILE_BYTES;
            const v4u v = *reinterpret_cast<const v4u *>(tile + lane * 16);
#pragma unroll
            for (int e = 0; e < 4; ++e) r.w[e] = v[e];
            return r;
        };
        auto product = [&](const Words &r, const Tile &t, v4f (&acc)[K]) {
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int k = 0; k < K; ++k)
                    acc[k] = mfma_signs(r.w[c * K + k], __builtin_shufflevector(t.half[c][k][0], t.half[c][k][1], 0, 1, 2, 3, 4, 5, 6, 7), acc[k], c22, scale_b);
        };
        // a quad of lanes holds the four terms of a token: its first lane files rows 4 qd .. 4 qd + 3
        auto file = [&](int p, const v4f (&acc)[K]) {
#pragma unroll
            for (int k = 0; k < K; ++k) {
                v4f v;
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = quad_sum(acc[k][r]);
                if ((col & 3) == 0)
                    *reinterpret_cast<v4f *>(lds + (((parity * MAXSLOT + s.slot0 + p) * CWAVES + wave) * PART + (k * T + (col >> 2)) * 16 + 4 * qd) * 4) = v;
            }
        };
        if (n <= M) {
            if (n > 0) request(0, n);
            // (pairs of row tiles where there are registers for them)
            const bool pairs = M <= 2 && 2 * s.CT <= TILES;
            int at = wrapped(ring + c0);
#pragma unroll 1
            for (int p = 0; p < s.P;) {
                const bool two = pairs && p + 1 < s.P;
                v4f acc0[K];
                Words w0[M];
#pragma unroll
                for (int k = 0; k < K; ++k) acc0[k] = (v4f){0.f, 0.f, 0.f, 0.f};
                wait_landed(base + (uint32_t)((p + (two ? 1 : 0)) * s.CT + c0 + n));
#pragma unroll
                for (int d = 0; d < M; ++d)
                    if (d < n) w0[d] = read_tile(at + d);
                at = wrapped(at + s.CT);
                if constexpr (M <= 2) {
                    if (two) {
                        v4f acc1[K];
                        Words w1[M];
#pragma unroll
                        for (int k = 0; k < K; ++k) acc1[k] = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int d = 0; d < M; ++d)
                            if (d < n) w1[d] = read_tile(at + d);
                        at = wrapped(at + s.CT);
#pragma unroll
                        for (int d = 0; d < M; ++d)
                            if (d < n)
#pragma unroll
                                for (int c = 0; c < 2; ++c)
#pragma unroll
                                    for (int k = 0; k < K; ++k) {
                                        const v8i t = __builtin_shufflevector(b[d].half[c][k][0], b[d].half[c][k][1], 0, 1, 2, 3, 4, 5, 6, 7);
                                        acc0[k] = mfma_signs(w0[d].w[c * K + k], t, acc0[k], c22, scale_b);
                                        acc1[k] = mfma_signs(w1[d].w[c * K + k], t, acc1[k], c22, scale_b);
                                    }
                        still_needs(row_of(p + 2));
                        file(p, acc0);
                        file(p + 1, acc1);
                        p += 2;
                        continue;
                    }
                }
#pragma unroll
                for (int d = 0; d < M; ++d)
                    if (d < n) product(w0[d], b[d], acc0);
                still_needs(row_of(p + 1));
                file(p, acc0);
                ++p;
            }
        } else {
            // (a row tile may be longer than the ring: what comes before this wavefront's columns is for others to give back)
            still_needs(row_of(0));
            int at = wrapped(ring + c0);
#pragma unroll 1
            for (int p = 0; p < s.P; ++p) {
                v4f acc[K];
#pragma unroll
                for (int k = 0; k < K; ++k) acc[k] = (v4f){0.f, 0.f, 0.f, 0.f};
                int here = at;
#pragma unroll 1
                for (int piece = 0; piece < n; piece += M) {
                    const int m = min(M, n - piece);
                    request(piece, m);
                    wait_landed(base + (uint32_t)(p * s.CT + c0 + piece + m));
#pragma unroll
                    for (int d = 0; d < M; ++d)
                        if (d < m) product(read_tile(here + d), b[d], acc);
                    here = wrapped(here + M);
                    still_needs(piece + m < n ? base + (uint32_t)(p * s.CT + c0 + piece + m) : row_of(p + 1));
                }
                file(p, acc);
                at = wrapped(at + s.CT);
            }
        }
    };
    auto run_segment = [&](const Segment &s, uint32_t base, int ring, int parity) {
        if (columns_of(s) <= 2) multiply(std::integral_constant<int, 2>(), s, base, ring, parity);
        else multiply(std::integral_constant<int, RESIDENT>(), s, base, ring, parity);
    };

    Work now = work[grp];
    uint32_t base = 0;                                       // the stage's first sign tile in the stream, and where it is in LDS
    int ring = 0;

    // ---- finishing: lane -> (row, token); up to six (reading op, path) pairs per row
    constexpr int PAIRS = MAX_CONS * K;
    const int row = lane & 15, tok = lane >> 4;
    // where a workgroup finishes few row tiles, several wavefronts share one: each works out the rows for itself and takes some of the pairs
    int fin_slot = 0, fin_part = 0, fin_parts = 1;
    // what finishing takes from the tables, asked for one stage ahead: values of the lane's row, and a card of words, one per lane: those of the
    // row tile's records in lanes 0 to 15, those of the stage after the next in lanes 16 to 31.  (In vector registers: a scalar load is waited for when its
    // result is put aside, and there are more of them than scalar registers)
    static_assert(sizeof(SlotRec) == 32 && sizeof(SlotExt) == 32 && sizeof(Work) == 64, "words of a card");
    uint32_t card = 0;
    float fin_g[K], fin_g_up[K], fin_h[PAIRS];
    auto word = [&](int i) -> uint32_t { return (uint32_t)__builtin_amdgcn_readlane((int)card, i); };
    auto word2 = [&](int i) -> uint64_t { return (uint64_t)word(i + 1) << 32 | word(i); };
    auto fetch = [&](const Work &w, int st) {
        // (worked out anew, so that no register holds what depends on it from stage to stage)
        int lane;
        asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane));
        const int row = lane & 15;
        const int n = max((int)w.n_fin, 1);
        fin_parts = n == 1 ? 8 : n == 2 ? 4 : n <= 4 ? 2 : 1;
        fin_slot = wave & (CWAVES / fin_parts - 1);
        fin_part = wave / (CWAVES / fin_parts);
        const size_t idx = (size_t)w.rec + (size_t)min(fin_slot, n - 1);
        const uint32_t *from = lane < 8 || (!BLK && lane < 16) ? reinterpret_cast<const uint32_t *>(slots + idx) + (lane & 7)
                               : lane < 16                     ? reinterpret_cast<const uint32_t *>(ext + idx) + (lane & 7)
                                                               : reinterpret_cast<const uint32_t *>(work + (size_t)min(st + 1, n_stages - 1) * n_groups + grp) + (lane & 15);
        card = *RB_GLOBAL(const uint32_t, from);
        const float *const v = vals + (idx * 16 + (size_t)row) * VALS_ROW;
#pragma unroll
        for (int k = 0; k < K; ++k) fin_g[k] = v[k];
#pragma unroll
        for (int m = 0; m < PAIRS; ++m) fin_h[m] = v[K + min(m * fin_parts + fin_part, PAIRS - 1)];
        if constexpr (BLK) {
            const float *const u = v + ((w.flags & WORK_GATED) ? GATED_SLOTS * 16 * VALS_ROW : 0);
#pragma unroll
            for (int k = 0; k < K; ++k) fin_g_up[k] = u[k];
        }
    };
    auto next_work = [&]() -> Work {
        union { uint32_t w[16]; Work work; } u;
#pragma unroll
        for (int i = 0; i < 16; ++i) u.w[i] = word(16 + i);
        return u.work;
    };
    fetch(now, 0);

#pragma unroll 1
    for (int st = 0; st < n_stages; ++st) {
        const int parity = st & 1;
        const bool have = fin_slot < now.n_fin, gated = BLK && (now.flags & WORK_GATED) != 0, norm = BLK && (now.flags & WORK_NORM) != 0;
        // ---- the time the slowest producer's stores need to land.  A workgroup without a part in the stage waits for twice that: the others take longer, and
        // what it asks for before they are done is stale in the L2 that it shares with some of them (one block of layers at three tokens, us without and with:
        // chains 2048 x 8192 35.9 and 28.1, 1280 x 5056 30.6 and 23.6, 3072 x 6144 31.1 and 28.1, a decoder block of 2048 x 8192 40.2 and 33.6; 64, 96 and 128
        // units for the built-in pause of 48 are the same within 2 %)
        if constexpr (LEFT_OUT) {
            const int pauses = now.P[0] == 0 ? (st + 1 < n_stages ? 2 : 0) : st > 0 && (now.flags & (WORK_DEP0 | WORK_DEP1)) != 0 ? 1 : 0;
            for (int i = 0; i < pauses * go_pause; ++i) __builtin_amdgcn_s_sleep(1);
        } else if (st > 0 && (now.flags & (WORK_DEP0 | WORK_DEP1)) != 0) {
            for (int i = 0; i < go_pause; ++i) __builtin_amdgcn_s_sleep(1);
        }
        // ---- decoder blocks: what comes from other workgroups' finishing wavefronts besides the operands.  Both kinds are marked "not yet
        // written" (all ones) before the launch and looked at until they are not.  The sums of squares of token `wave`:
        constexpr int SSQ = 4;
        [[maybe_unused]] uint32_t squares[SSQ];
        [[maybe_unused]] uint32_t added = 0;
        [[maybe_unused]] const bool sums = norm && wave < tokens;
        [[maybe_unused]] const uint32_t rec_out = BLK ? word(5) : 0, rec_flags = BLK ? word(6) : 0;
        [[maybe_unused]] const uint64_t resid = BLK ? word2(8) : 0;
        [[maybe_unused]] const int kind = BLK && have && row < (int)(rec_flags & 0xffu) && tok < tokens ? (int)(rec_flags >> 16 & 0xffu) : RESID_NONE;
        [[maybe_unused]] const uint32_t *const ssq_in = reinterpret_cast<const uint32_t *>(up0 + (uint64_t)now.ssq_in * 256) + (size_t)wave * now.n_part;
        [[maybe_unused]] auto square = [&](uint32_t i) -> uint32_t {
            return i < now.n_part ? __hip_atomic_load(RB_GLOBAL(const uint32_t, ssq_in) + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
        };
        [[maybe_unused]] auto copy_of = [&]() -> uint32_t {
            return __hip_atomic_load(RB_GLOBAL(const uint32_t, resid) + (size_t)tok * rec_out + row, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        };
        if constexpr (BLK) {
            if (sums)
#pragma unroll
                for (int i = 0; i < SSQ; ++i) squares[i] = square((uint32_t)(lane + 64 * i));
            if (kind == RESID_COPY) added = copy_of();
            if (kind == RESID_CALLER) added = RB_GLOBAL(const uint16_t, resid)[(size_t)tok * rec_out + row];
        }

#pragma unroll 1
        for (int n = 0; n < 2; ++n) {
            const Segment s = n == 0 ? first_of(now) : second_of(now);
            if (s.P == 0) break;
            run_segment(s, base, ring, parity);
            const int count = s.P * s.CT;
            base += (uint32_t)count;
            ring += count;
            while (ring >= TILES) ring -= TILES;
        }

        if constexpr (BLK) {
            if (sums) {
                float total = 0.f;
                bool missing;
                uint32_t looks = 0;
                do {
                    missing = false;
                    total = 0.f;
#pragma unroll
                    for (int i = 0; i < SSQ; ++i) {
                        missing |= squares[i] == 0xffffffffu;
                        total += __uint_as_float(squares[i]);
                    }
                    for (uint32_t i = SSQ * 64; i < now.n_part; i += 64) {
                        const uint32_t v = square((uint32_t)lane + i);
                        missing |= v == 0xffffffffu;
                        total += __uint_as_float(v);
                    }
                    missing = __ballot(missing) != 0ull && !failed;
                    if (missing) {
                        __builtin_amdgcn_s_sleep(8);
                        if (looks > QUICK_LOOKS) __builtin_amdgcn_s_sleep(56);
                        ++looks;
#pragma unroll
                        for (int i = 0; i < SSQ; ++i) squares[i] = square((uint32_t)(lane + 64 * i));
                    }
                } while (missing && looks < MAX_LOOKS);
                if (missing) give_up(GAVE_UP_BLOCK);
#pragma unroll
                for (int m = 1; m < 64; m <<= 1) total += __shfl_xor(total, m);
                const float rinv = rsqrtf(total * now.inv_n + eps);
                if (lane == 0) asm volatile("ds_write_b32 %0, %1" : : "v"(lds_at(Lds::RINV_OFF + (parity * 4 + wave) * 4)), "v"(rinv) : "memory");
            }
            uint32_t looks = 0;
            while (!failed && looks < MAX_LOOKS && __ballot(kind == RESID_COPY && added == 0xffffffffu) != 0ull) {
                __builtin_amdgcn_s_sleep(8);
                if (looks > QUICK_LOOKS) __builtin_amdgcn_s_sleep(56);
                ++looks;
                if (kind == RESID_COPY) added = copy_of();
            }
            if (looks == MAX_LOOKS) give_up(GAVE_UP_BLOCK);
        }
        // ---- the partial sums of the stage are in LDS when all have got here (the loading wavefront takes no part).  In place one of the wavefronts
        // that finish the same rows stores over what all of them add: it has arrived with each before any comes by here (the compiler waits for
        // a loaded value that a statement takes)
        if constexpr (BLK) asm volatile("" : "+v"(added) : : "memory");
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (lane == 0) lds_add(lds_at(Lds::ARRIVED_OFF), 1u);
        while ((int)(lds_read(lds_at(Lds::ARRIVED_OFF)) - (uint32_t)(CWAVES * (st + 1))) < 0) {}
        if (have) {
            const uint64_t y_at = word2(0);
            const uint32_t up_at[MAX_CONS] = {word(2), word(3), word(4)};
            const int out = (int)word(5), rows = (int)(word(6) & 0xffu), n_pairs = (int)(word(6) >> 8 & 0xffu) * K;
            const bool active = row < rows && tok < tokens;
            auto row_sum_of = [&](int slot, const float (&g)[K]) -> float {
                const uint32_t from = lds_at(((parity * MAXSLOT + slot) * CWAVES * PART + tok * 16 + row) * 4);
                float s[K];
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    float v[CWAVES];
                    static_assert(CWAVES == 8, "eight partial sums");
                    asm volatile("ds_read_b32 %0, %8 offset:%9\n\t"
                                 "ds_read_b32 %1, %8 offset:%10\n\t"
                                 "ds_read_b32 %2, %8 offset:%11\n\t"
                                 "ds_read_b32 %3, %8 offset:%12\n\t"
                                 "ds_read_b32 %4, %8 offset:%13\n\t"
                                 "ds_read_b32 %5, %8 offset:%14\n\t"
                                 "ds_read_b32 %6, %8 offset:%15\n\t"
                                 "ds_read_b32 %7, %8 offset:%16\n\t"
                                 "s_waitcnt lgkmcnt(0)"
                                 : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7])
                                 : "v"(from + k * (T * 64)), "n"(0), "n"(PART * 4), "n"(PART * 8), "n"(PART * 12), "n"(PART * 16), "n"(PART * 20),
                                   "n"(PART * 24), "n"(PART * 28)
                                 : "memory");
                    s[k] = 0.f;
#pragma unroll
                    for (int w = 0; w < CWAVES; ++w) s[k] += v[w];
                }
                return path_sum(g[0], s[0], g[1], s[1]);
            };
            float y = row_sum_of(fin_slot, fin_g);
            if constexpr (BLK) {
                float rinv = 1.f;
                if (norm) asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(rinv) : "v"(lds_at(Lds::RINV_OFF + (parity * 4 + (tok < tokens ? tok : 0)) * 4)) : "memory");
                y *= rinv;                                    // the input was x / rms(x) (.) w
                if (gated) y = y / (1.f + __expf(-y)) * (row_sum_of(GATED_SLOTS + fin_slot, fin_g_up) * rinv);
                if (kind != RESID_NONE) y += __half2float(__ushort_as_half((unsigned short)added));
            }
            const _Float16 y16 = (_Float16)y;                 // round to nearest even
            const float yf = active ? (float)y16 : 0.f;
            if constexpr (BLK) {
                const uint32_t ssq_at = word(10), rcopy_at = word(12);
                if (rcopy_at && active && fin_part == 0)
                    store_sc1_u32((uint64_t)up0 + ((uint64_t)rcopy_at + (uint32_t)(tok * out + row)) * 4, (uint32_t)__builtin_bit_cast(uint16_t, y16));
                if (ssq_at) {
                    // this row tile's sum of squares, for the ops that normalise what they read
                    const float sq = row_sum(yf * yf);
                    if (row == 0 && fin_part == 0 && tok < tokens) store_sc1_u32((uint64_t)up0 + ((uint64_t)ssq_at + (uint32_t)(tok * (int)word(11))) * 4, __float_as_uint(sq));
                }
            }
            // ---- expanded input of the ops that read y next: the term bytes of the 16 rows of a
            // (token, path), one word per lane of a 16-lane row, are transposed in registers into one
            // 16-byte group per term, which lanes 0..3 of the row store.  Rows beyond the end of the
            // matrix and tokens that are not there give zero bytes.
#pragma unroll
            for (int m = 0; m < PAIRS; ++m)
                if (m * fin_parts + fin_part < n_pairs) {
                    const int pair = m * fin_parts + fin_part, c = pair / K, k = pair % K;
                    const v4i bytes = transpose_16x4_bytes(active ? expand4(fin_h[m] * yf) : 0u);
                    const uint32_t base = c == 0 ? up_at[0] : c == 1 ? up_at[1] : up_at[2];
                    const uint8_t *const to = up0 + ((uint64_t)base + (uint32_t)(k * C + 4 * tok + row)) * 16;
                    if (row < 4) asm volatile("global_store_dwordx4 %0, %1, off sc1" : : "v"(to), "v"(bytes) : "memory");
                }
            if (y_at && active && fin_part == 0) RB_GLOBAL(_Float16, y_at)[(size_t)tok * out + row] = y16;
        }
        // ---- the tables of the next stage, in the time that the outputs need to get there
        now = next_work();
        fetch(now, st + 1);
    }
    if (lane == 0 && waited != 0) __hip_atomic_fetch_add(RB_GLOBAL(uint32_t, error) + 1, waited, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ------------------------------------------------------------------ host ---
static Layout make_layout(int n_ops, int n_stages, int G, size_t n_records, size_t up_total, bool block = false, size_t aux_poison = 0, size_t aux_rest = 0)
{
    Layout L;
    size_t o = 0;
    L.ops = o; o += sizeof(Op) * (size_t)n_ops;
    o = align_up(o, 128); L.stages = o; o += sizeof(Stage) * (size_t)n_stages;
    o = align_up(o, 128); L.error = o; o += 128;
    L.which = o; o += align_up(sizeof(int) * MAX_EXPAND, 128);
    o = align_up(o, 128); L.work = o; o += sizeof(Work) * (size_t)n_stages * (size_t)G;
    o = align_up(o, 128); L.slots = o; o += sizeof(SlotRec) * n_records;
    o = align_up(o, 128); L.vals = o; o += VALS_RECORD_BYTES * n_records;
    L.ext = o;
    if (block) { o = align_up(o, 128); L.ext = o; o += sizeof(SlotExt) * n_records; }
    o = align_up(o, 256); L.up = o; o += up_total;
    L.aux = o; L.aux_poison = 0;
    if (block) {
        o = align_up(o, 256); L.aux = o; o += align_up(aux_poison, 256) + align_up(aux_rest, 256);
        L.aux_poison = align_up(aux_poison, 256);
    }
    L.total = align_up(o, 256);
    return L;
}

size_t plan_workspace_bytes(const rb_layer *layers, int n_layers, int n_ops, int tokens, bool block)
{
    // upper bound: every op could use the widest layer
    size_t up_max = 0;
    int G = device_groups(), slots = 1;
    if (G <= 0) G = 1024;  // no device to ask: a bound on compute units
    for (int l = 0; l < n_layers; ++l) {
        up_max = std::max(up_max, up_bytes(layers[l].in));
        slots = std::max(slots, (row_tiles(layers[l].out) + G - 1) / G);
    }
    if (block) slots = std::max(slots, GATED_SLOTS);     // (gate and up are two ops)
    return make_layout(n_ops, n_ops, G, (size_t)n_ops * (size_t)G * (size_t)std::min(slots, MAXSLOT), align_up(up_max, 256) * (size_t)n_ops, block,
                       block ? block_aux_bound(layers, n_layers, tokens) * (size_t)n_ops : 0, 0)
        .total;
}

// Host record of a prepared plan, keyed by the workspace that holds its device part.
struct Prepared {
    Layout lay;
    int n_ops = 0, n_stages = 0, G = 0, tokens = 0, max_expand_in = 0, n_expand = 0;
    bool chained = false;                   // some op reads what another op of the launch writes
    bool block = false;                     // a decoder block: the kernel form with the epilogues
    bool ext_norm = false;                  // some op normalises an input from outside
    bool aside = false;                     // some op adds what has to be put aside before the launch
    bool left_out = false;                  // some stage has fewer row tiles than there are workgroups
    float eps = 0.f;
    // host memory the plan's tables are copied from: pageable, so it must outlive the queued copies
    std::shared_ptr<std::vector<uint8_t>> blob;
    std::shared_ptr<std::vector<int>> which;
};
static std::mutex g_mutex;
static std::map<const void *, Prepared> g_prepared;
constexpr int STAGE_TILES = 96;             // sign tiles that a workgroup multiplies in the time that a stage takes besides

int prepare(const rb_layer *layers, const PlanOp *sops, const OpLinks *links, int n_ops, uint16_t *const *bufs,
                       const uint16_t *const *norm_w, float eps, bool block, int tokens, void *workspace,
                       size_t workspace_bytes_, hipStream_t stream)
{
    const int G = device_groups();
    if (G <= 0) return RB_ERR_HIP;

    // ---- ops, consumers, stages
    std::vector<Op> ops((size_t)n_ops);
    std::vector<int> expand_list;
    size_t up_total = 0;
    std::vector<size_t> up_off((size_t)n_ops);
    for (int n = 0; n < n_ops; ++n) {
        const rb_layer &L = layers[sops[n].layer];
        Op &o = ops[(size_t)n];
        std::memset(&o, 0, sizeof(Op));
        o.bits = static_cast<const uint32_t *>(L.bits);
        o.g = L.g; o.h = L.h;
        o.x = bufs[sops[n].src];
        o.y = sops[n].dst >= 0 && links[n].stores ? bufs[sops[n].dst] : nullptr;
        o.norm_w = sops[n].norm >= 0 ? norm_w[sops[n].norm] : nullptr;
        o.out = L.out; o.in = L.in;
        o.RT = row_tiles(L.out); o.CT = col_tiles(L.in);
        up_off[(size_t)n] = up_total;
        up_total += align_up(up_bytes(L.in), 256);
        const OpLinks &l = links[n];
        o.dep = l.producer;
        if (o.norm_w) o.n_part = (L.in + 15) / 16;
        if (sops[n].add >= 0) {
            o.resid_kind = l.addend >= 0 ? RESID_COPY : RESID_CALLER;
            if (l.aside) o.resid_src = bufs[sops[n].add];
            else if (l.addend < 0) o.resid = bufs[sops[n].add];
        }
        o.n_cons = l.n_cons;
        std::copy(l.cons, l.cons + l.n_cons, o.cons);
        if (l.producer < 0) expand_list.push_back(n);
    }
    std::vector<Stage> stages;
    size_t n_records = 0;
    for (int op0 = 0; op0 < n_ops;) {
        Stage s{};
        s.op0 = op0;
        s.norm = ops[(size_t)op0].norm_w != nullptr;
        int ct_max = 0;
        for (int n = op0; n < n_ops && s.nops < MAX_STAGE_OPS; ++n) {
            bool conflict = false;
            for (int m = op0; m < n; ++m) {
                if (sops[m].dst < 0 || sops[n].dst < 0) continue;
                if (sops[m].dst == sops[n].src || sops[m].dst == sops[n].dst || sops[m].src == sops[n].dst ||
                    sops[m].dst == sops[n].add || sops[m].add == sops[n].dst)
                    conflict = true;
            }
            const Op &o = ops[(size_t)n];
            if ((o.RT + G - 1) / G > MAXSLOT) return RB_ERR_UNSUPPORTED;
            if (sops[n].role == ROLE_GATE) {
                // gate and up: a stage of their own; the row tiles of the two are dealt alike
                if (n > op0) break;
                if ((o.RT + G - 1) / G > GATED_SLOTS) return RB_ERR_UNSUPPORTED;
                s.nops = 2;
                s.gated = 1;
                s.tiles = s.rt[0] = s.rt[1] = o.RT;
                break;
            }
            // one root mean square per token and stage: normalised ops share one only if they read the same
            if ((o.norm_w != nullptr) != (s.norm != 0) || (s.norm && (sops[n].src != sops[op0].src || o.dep != ops[(size_t)op0].dep))) conflict = true;
            // a workgroup's share lies in at most two ops: those between the first and the last are no shorter than a share
            const int share = (s.tiles + o.RT + G - 1) / G, longest = std::max(ct_max, o.CT);
            for (int i = 1; i < s.nops; ++i)
                if (s.rt[i] < share) conflict = true;
            if (conflict || share > MAXSLOT) break;
            // Row tiles are dealt by number, so longer rows among shorter ones make some workgroups late: ops of other widths come along only where that is no
            // more than a stage for each width would take (us of ops that read what the caller has, three tokens, together and apart: 4096 x 4096, two
            // 11008 x 4096 and 4096 x 11008 49.5 and 23.8; 56 ops of 2048 x 5504 blocks, which leave half of the workgroups out, 62 and 98).  With a row tile or less for each
            // workgroup neither is good: such plans are for the step lists, which deal each op by itself (14 pairs of 11008 x 4096 and 4096 x 11008 213 there, 307 and 228
            // here, 28 ops of 2304 x 9216 blocks 66, 144 and 72; not 28 of 3584 x 9472, 100, 89 and 93)
            int by_width = -STAGE_TILES;
            bool uneven = false;
            for (int i = 0; i <= s.nops; ++i) {
                const Op &first = ops[(size_t)(op0 + i)];
                int rt = 0, before = 0;
                for (int j = 0; j <= s.nops; ++j)
                    if (ops[(size_t)(op0 + j)].CT == first.CT) { rt += ops[(size_t)(op0 + j)].RT; before += j < i; }
                if (before == 0) by_width += STAGE_TILES + (rt + G - 1) / G * first.CT;
                if (first.CT != o.CT && 2 * first.RT > G && 2 * o.RT > G) {
                    if (std::min(first.RT, o.RT) <= G) return RB_ERR_UNSUPPORTED;
                    uneven = true;
                }
            }
            if (uneven || share * longest > by_width) break;
            s.rt[s.nops++] = o.RT;
            s.tiles += o.RT;
            ct_max = longest;
        }
        s.n_slots = (s.tiles + G - 1) / G + (s.gated ? GATED_SLOTS : 0);
        s.rec0 = (uint32_t)n_records;
        n_records += (size_t)G * (size_t)s.n_slots;
        stages.push_back(s);
        op0 += s.nops;
    }
    Prepared pr;
    pr.n_ops = n_ops; pr.n_stages = (int)stages.size(); pr.G = G; pr.tokens = tokens;
    pr.n_expand = (int)expand_list.size();
    for (const Stage &s : stages) pr.left_out = pr.left_out || s.tiles < G;
    for (int n : expand_list) pr.max_expand_in = std::max(pr.max_expand_in, ops[(size_t)n].in);
    for (int n = 0; n < n_ops; ++n) pr.chained = pr.chained || ops[(size_t)n].dep >= 0 || links[n].addend >= 0;
    // decoder blocks: what finishing wavefronts hand to each other (marked unwritten before every
    // launch), then the sums of squares of inputs from outside and what is put aside
    std::vector<size_t> ssq_off((size_t)n_ops, 0), rcopy_off((size_t)n_ops, 0), ext_off((size_t)n_ops, 0), aside_off((size_t)n_ops, 0);
    size_t aux_poison = 0, aux_rest = 0;
    for (int n = 0; n < n_ops && block; ++n) {
        if (links[n].squares) { ssq_off[(size_t)n] = aux_poison; aux_poison += align_up((size_t)ops[(size_t)n].RT * 16, 256); }
        if (links[n].copied) { rcopy_off[(size_t)n] = aux_poison; aux_poison += align_up((size_t)tokens * ops[(size_t)n].out * 4, 256); }
        if (ops[(size_t)n].norm_w && ops[(size_t)n].dep < 0) {
            ext_off[(size_t)n] = aux_rest;
            aux_rest += align_up((size_t)ops[(size_t)n].n_part * 16, 256);
            pr.ext_norm = true;
        }
        if (links[n].aside) {
            aside_off[(size_t)n] = aux_rest;
            aux_rest += align_up((size_t)tokens * ops[(size_t)n].out * 2, 256);
            pr.aside = true;
        }
    }
    pr.block = block;
    // (offsets of the tables hold 32 bits)
    if (n_records > 0xffffffffull || up_total + aux_poison + aux_rest > 0x3fffffff0ull) return RB_ERR_UNSUPPORTED;
    pr.lay = make_layout(n_ops, pr.n_stages, G, n_records, up_total, block, aux_poison, aux_rest);
    pr.eps = eps;
    const Layout &lay = pr.lay;
    if (workspace_bytes_ < lay.total) return RB_ERR_WORKSPACE;
    uint8_t *ws = static_cast<uint8_t *>(workspace);
    for (int n = 0; n < n_ops; ++n) ops[(size_t)n].up = ws + lay.up + up_off[(size_t)n];
    for (int n = 0; n < n_ops && block; ++n) {
        Op &o = ops[(size_t)n];
        if (links[n].squares) o.ssq_out = reinterpret_cast<float *>(ws + lay.aux + ssq_off[(size_t)n]);
        if (links[n].copied) o.rcopy = reinterpret_cast<uint32_t *>(ws + lay.aux + rcopy_off[(size_t)n]);
    }
    for (int n = 0; n < n_ops && block; ++n) {
        Op &o = ops[(size_t)n];
        if (o.norm_w)
            o.ssq_in = o.dep >= 0 ? ops[(size_t)o.dep].ssq_out
                                  : reinterpret_cast<const float *>(ws + lay.aux + lay.aux_poison + ext_off[(size_t)n]);
        if (links[n].addend >= 0) o.resid = ops[(size_t)links[n].addend].rcopy;
        if (links[n].aside) o.resid = ws + lay.aux + lay.aux_poison + aside_off[(size_t)n];
    }

    // ---- upload: stream-ordered copies out of host memory that the plan's record keeps alive
    pr.blob = std::make_shared<std::vector<uint8_t>>(lay.error, (uint8_t)0);
    std::vector<uint8_t> &blob = *pr.blob;
    std::memcpy(blob.data() + lay.ops, ops.data(), sizeof(Op) * (size_t)n_ops);
    std::memcpy(blob.data() + lay.stages, stages.data(), sizeof(Stage) * (size_t)pr.n_stages);
    pr.which = std::make_shared<std::vector<int>>(expand_list);
    const int *which = pr.which->data();
    if (hipMemcpyAsync(ws, blob.data(), lay.error, hipMemcpyHostToDevice, stream) != hipSuccess) return RB_ERR_HIP;
    if (!expand_list.empty() &&
        hipMemcpyAsync(ws + lay.which, which, sizeof(int) * expand_list.size(), hipMemcpyHostToDevice, stream) !=
            hipSuccess)
        return RB_ERR_HIP;
    {
        std::lock_guard<std::mutex> lock(g_mutex);
        g_prepared[workspace] = pr;
    }
    hipLaunchKernelGGL(prep_kernel, dim3(n_ops), dim3(256), 0, stream, reinterpret_cast<Op *>(ws + lay.ops),
                       reinterpret_cast<uint32_t *>(ws + lay.error));
    hipLaunchKernelGGL(link_kernel, dim3(pr.n_stages, (G + LINK_GROUPS - 1) / LINK_GROUPS), dim3(256), 0, stream,
                       reinterpret_cast<const Op *>(ws + lay.ops), reinterpret_cast<const Stage *>(ws + lay.stages), G,
                       reinterpret_cast<Work *>(ws + lay.work), reinterpret_cast<SlotRec *>(ws + lay.slots),
                       reinterpret_cast<float *>(ws + lay.vals), block ? reinterpret_cast<SlotExt *>(ws + lay.ext) : nullptr, ws + lay.up);
    return hipGetLastError() == hipSuccess ? RB_OK : RB_ERR_HIP;
}

// RB_ERR_UNSUPPORTED: the workspace holds no plan of this kind
int launch(void *workspace, size_t workspace_bytes_, int pause, hipStream_t stream)
{
    Prepared pr;
    {
        std::lock_guard<std::mutex> lock(g_mutex);
        const auto it = g_prepared.find(workspace);
        if (it == g_prepared.end()) return RB_ERR_UNSUPPORTED;
        pr = it->second;
    }
    if (workspace_bytes_ < pr.lay.total) return RB_ERR_WORKSPACE;
    uint8_t *ws = static_cast<uint8_t *>(workspace);
    const Layout &lay = pr.lay;
    Op *d_ops = reinterpret_cast<Op *>(ws + lay.ops);
    const int n_poison = pr.chained ? (pr.n_ops + (lay.aux_poison ? 1 : 0)) * POISON_SPLIT : 0;
    const int ex = (pr.max_expand_in / 16 * K + 255) / 256, ey = pr.tokens;
    const int n_expand_groups = pr.n_expand > 0 ? ex * ey * pr.n_expand : 0;
    const int n_ssq_groups = pr.ext_norm ? pr.n_expand * ey : 0, n_aside_groups = pr.aside ? pr.n_ops * ASIDE_SPLIT : 0;
    if (n_poison + n_expand_groups + n_ssq_groups + n_aside_groups > 0)
        hipLaunchKernelGGL(before_kernel, dim3((unsigned)(n_poison + n_expand_groups + n_ssq_groups + n_aside_groups)), dim3(256), 0, stream, d_ops,
                           pr.n_ops, reinterpret_cast<const int *>(ws + lay.which), n_poison, n_expand_groups, ex, ey, n_ssq_groups,
                           reinterpret_cast<uint4 *>(ws + lay.aux), lay.aux_poison / 16);
    const int go_pause = pause < 0 ? GO_PAUSE : pause / 64;          // s_sleep units
    auto launch_form = [&](auto kernel) -> int {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, Lds::BYTES) != hipSuccess)
            return RB_ERR_HIP;
        hipLaunchKernelGGL(kernel, dim3(pr.G), dim3(THREADS), Lds::BYTES, stream, reinterpret_cast<const Work *>(ws + lay.work), reinterpret_cast<const SlotRec *>(ws + lay.slots),
                           reinterpret_cast<const float *>(ws + lay.vals), reinterpret_cast<const SlotExt *>(ws + lay.ext), ws + lay.up,
                           reinterpret_cast<uint32_t *>(ws + lay.error), pr.n_stages, pr.tokens, go_pause, pr.eps);
        return RB_OK;
    };
    const int rc = pr.block ? (pr.left_out ? launch_form(flow_kernel<true, true>) : launch_form(flow_kernel<true, false>))
                            : (pr.left_out ? launch_form(flow_kernel<false, true>) : launch_form(flow_kernel<false, false>));
    if (rc != RB_OK) return rc;
    return hipGetLastError() == hipSuccess ? RB_OK : RB_ERR_HIP;
}

// where a plan's marks are (gave up a wait; tiles waited for); null: no plan of this kind
const void *marks(const void *workspace)
{
    std::lock_guard<std::mutex> lock(g_mutex);
    const auto it = g_prepared.find(workspace);
    return it == g_prepared.end() ? nullptr : static_cast<const uint8_t *>(workspace) + it->second.lay.error;
}

void forget(const void *workspace)
{
    std::lock_guard<std::mutex> lock(g_mutex);
    g_prepared.erase(workspace);
}

}  // namespace flow
}  // namespace rb
