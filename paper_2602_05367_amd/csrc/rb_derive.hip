// Initialisation of the paths from a full-precision weight (Section 4.3, Alg. 1): Iterative
// Residual SVID on the preconditioned weight W' = rows (.) W (.) cols (Eq. init-calib).
//
//   What_i = 0;  for t = 1..T_max, for i = 1..K:
//       R_i = W' - sum_{j != i} What_j        (Eq. init-iter; paths j < i of this sweep, j > i of the last)
//       B_i = sign(R_i);  (sigma, a, b) = leading singular triplet of |R_i|
//       g_i' = sqrt(sigma) a,  h_i' = sqrt(sigma) b;  What_i = g_i' (.) B_i (.) h_i'
//   g_i = g_i' / rows,  h_i = h_i' / cols
//
// Everything is fp64 (the sign of a residual decides a stored bit).  No residual and no What_i is
// ever materialised: a path is its packed signs and two vectors, and every pass recomputes R_i
// from W (4 bytes per weight) and the other paths (a bit and two cached scale values each), so a
// pass is bound by the HBM read of W.  The singular triplet comes from a power iteration from the
// all-ones vector (the matrix is non-negative): a = |R| b, c = |R|^T a.  One reading of W serves both where a row fits the registers
// of a workgroup (one_pass_kernel); else there are two passes, by rows (four rows
// per workgroup) and by columns (slices of rows, partial sums added in slice order).  In all of them a lane takes
// four consecutive columns, one 16-byte load of W.  a is left at its length and its norm taken
// out of c: with b of length 1, sigma = ||c|| and the next b is c / ||c||.  After the last iteration one more pass by rows gives the last |R| b and the
// signs of R_i.  The error after an update, term by term (as ||R_i||^2 - sigma^2 it would come out of the same pass, but with
// a digit less: 3.6e-15 off where the terms are 1e-16), is found by the pass after the iteration while it holds a row of R, or, by two passes, by
// the first pass of the next update on the way: its R less the path that it leaves out.  Every sum has a fixed order.  The
// iteration's stopping rule is evaluated on the device.  Where one reading serves both passes, the device goes on to the next update by itself and the host
// looks a few times in all how far it has come; else it reads a flag per update when it expects the iteration to have finished.  So the call synchronises.
//
// Measured, 4096 x 11008, two paths, five sweeps (ten updates of four iterations): 2.3 to 2.45 ms (2.6 to 2.8 with a look at the flag after every update and launches of its
// start and end; 3.1 to 3.2 with launches of their own for b and for the errors; 3.9 with
// two passes in every iteration; 5.1 before those): an iteration is one pass of 40 to 42 us and 5.7 for the sums, the pass after it 45 to 47 (by rows, without the errors, 35).
// By two passes: 31 us each, the sums and the normalisation 12.  180 MB of W in
// 31 us are 5.8 TB/s, what a plain read of as much out of the memory-side cache reaches (6.0); of the 42 us some 7 are b and the
// columns' values at the start and 3 the 22 MB of sums at the end.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <type_traits>

#include "rabit.h"
#include "rb_device.h"
#include "rb_internal.h"
#include "rb_walk.h"

namespace rb {
namespace derive {

constexpr int ROW_SLICE = 32;          // rows one workgroup of the column pass walks (twice that where the workspace is the smaller)
constexpr int MAX_SLICES = 65535;
constexpr int ROWS = 4;                // rows one workgroup of the row pass takes
constexpr int MAX_ITER = 200;
constexpr int ONE_PASS_MIN_ROWS = 1024, ONE_PASS_MIN_COLS = 2048;
constexpr double TOL_SIGMA = 1e-13, TOL_B = 1e-10;

// W and the J paths that a pass subtracts
template <int J> struct Problem {
    const float *W;
    const double *rows, *cols;         // preconditioning factors (nullptr: 1)
    const uint32_t *packed[J + 1];     // [out][in/32] each (the last one of a first pass: the path itself as the last sweep left it)
    const double *g[J + 1], *h[J + 1]; // [out], [in]: g', h' of the preconditioned domain
    int out, in;
};

struct Scalars {
    double sigma;       // the iteration's current estimate
    double na;          // norm of |R| b
    double db;          // norm of the last change of b
    int done;           // the stopping rule held (or the matrix is zero); WALKED: nothing is left to do
    int iters;
    int t, i;           // the update that this belongs to (one_pass_kernel)
};
constexpr int WALKED = 2;

// sum over the wavefront, in every lane (every lane must be active): data-parallel moves inside a row of 16 lanes, register swaps
// beyond
__device__ __forceinline__ double over_wave(double v)
{
    auto both = [](double v, auto move) {
        const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
        return __builtin_bit_cast(double, (unsigned long long)move((uint32_t)(u >> 32)) << 32 | move((uint32_t)u));
    };
    v += both(v, [](uint32_t w) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, 0xB1, 0xf, 0xf, false); });      // quad_perm [1,0,3,2]
    v += both(v, [](uint32_t w) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, 0x4E, 0xf, 0xf, false); });      // quad_perm [2,3,0,1]
    v += both(v, [](uint32_t w) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, 0x141, 0xf, 0xf, false); });     // row_half_mirror
    v += both(v, [](uint32_t w) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, 0x140, 0xf, 0xf, false); });     // row_mirror
    auto swap_add = [](double v, auto swap) {
        const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
        const auto low = swap((uint32_t)u), high = swap((uint32_t)(u >> 32));
        return __builtin_bit_cast(double, (unsigned long long)high[0] << 32 | low[0]) + __builtin_bit_cast(double, (unsigned long long)high[1] << 32 | low[1]);
    };
    v = swap_add(v, [](uint32_t w) { return __builtin_amdgcn_permlane16_swap(w, w, false, false); });
    return swap_add(v, [](uint32_t w) { return __builtin_amdgcn_permlane32_swap(w, w, false, false); });
}

// sum over a workgroup of `waves` wavefronts in a fixed order, in every thread; red has a slot per wavefront
__device__ __forceinline__ double group_sum(double v, double *red, int waves)
{
    v = over_wave(v);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = 0.0;
    for (int w = 0; w < waves; ++w) s += red[w];
    __syncthreads();
    return s;
}

__global__ __launch_bounds__(256) void start_kernel(double *b, int in, Scalars *sc)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < in) b[i] = 1.0 / sqrt((double)in);
    if (i == 0) {
        sc->sigma = 0.0; sc->na = 0.0; sc->db = 0.0; sc->done = 0; sc->iters = 0;
    }
}

// What a step of a pass fetches: four consecutive columns of ROWS rows of W and the sign words they lie in, for N paths.
// No branch around any of it (rows past the last one: the last one): with the path left out found at run time the
// compiler put a branch and a full wait around every sign word, which took a quarter of the time of a pass
template <int N> struct Piece {
    float4 w[ROWS];
    uint32_t bits[ROWS][N + 1];
};
template <int J, int N>
__device__ __forceinline__ void fetch(const Problem<J> &p, int r, int r_last, int c, Piece<N> &to)
{
    const int W32 = p.in / 32;
#pragma unroll
    for (int u = 0; u < ROWS; ++u) {
        const int row = min(r + u, r_last);
        to.w[u] = *reinterpret_cast<const float4 *>(p.W + (size_t)row * p.in + c);
#pragma unroll
        for (int j = 0; j < N; ++j) to.bits[u][j] = p.packed[j][(size_t)row * W32 + (c >> 5)];
    }
}
// four consecutive values of a vector of doubles
__device__ __forceinline__ void four(const double *v, int c, double (&to)[4])
{
    const double2 a = *reinterpret_cast<const double2 *>(v + c), b = *reinterpret_cast<const double2 *>(v + c + 2);
    to[0] = a.x; to[1] = a.y; to[2] = b.x; to[3] = b.y;
}
// What a step shares of the columns, which is read once for ROWS rows (28 bytes through the caches for the 4 bytes of a weight
// with one row at a time): the factors and the paths' h
template <int N> struct Columns { double f[4], h[N + 1][4]; };
template <int J, int N> __device__ __forceinline__ void fetch_columns(const Problem<J> &p, int c, Columns<N> &to)
{
    to.f[0] = to.f[1] = to.f[2] = to.f[3] = 1.0;
    if (p.cols) four(p.cols, c, to.f);
#pragma unroll
    for (int j = 0; j < N; ++j) four(p.h[j], c, to.h[j]);
}
// and of the rows
template <int N> struct Rows { double rows[ROWS], g[ROWS][N + 1]; };
template <int J, int N> __device__ __forceinline__ void fetch_rows(const Problem<J> &p, int r, int r_last, Rows<N> &to)
{
#pragma unroll
    for (int u = 0; u < ROWS; ++u) {
        const int row = min(r + u, r_last);
#pragma unroll
        for (int j = 0; j < N; ++j) to.g[u][j] = p.g[j][row];
        to.rows[u] = p.rows ? p.rows[row] : 1.0;
    }
}
// v -= g B h for path j: the sign of g B is the bit of the column put on top of g
template <int N>
__device__ __forceinline__ void subtract(const Piece<N> &piece, const Columns<N> &cols, const Rows<N> &rows, int j, int c, double (&v)[ROWS][4])
{
#pragma unroll
    for (int u = 0; u < ROWS; ++u) {
        const uint32_t bits = piece.bits[u][j] >> (c & 31);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const unsigned long long flip = (unsigned long long)(bits << (31 - e) & 0x80000000u) << 32;
            v[u][e] -= __builtin_bit_cast(double, __builtin_bit_cast(unsigned long long, rows.g[u][j]) ^ flip) * cols.h[j][e];
        }
    }
}
// R[r ..][c .. c + 3] = rows W cols - the J paths
template <int J, int N>
__device__ __forceinline__ void residuals(const Problem<J> &p, const Piece<N> &piece, const Columns<N> &cols, const Rows<N> &rows, int c, double (&v)[ROWS][4])
{
#pragma unroll
    for (int u = 0; u < ROWS; ++u) {
        v[u][0] = (double)piece.w[u].x; v[u][1] = (double)piece.w[u].y; v[u][2] = (double)piece.w[u].z; v[u][3] = (double)piece.w[u].w;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[u][e] = rows.rows[u] * v[u][e] * cols.f[e];
    }
#pragma unroll
    for (int j = 0; j < J; ++j) subtract<N>(piece, cols, rows, j, c, v);
}

// a[r] = sum_c |R[r][c]| b[c], its square by workgroup; ROWS rows per workgroup, 1024 columns per step, the next step's
// fetches in flight.  FINAL (after the iteration): also the signs of R (sign(0) = +1;
// 32 columns per word, bit b = column 32 w + b, 1 means -1; nobody reads the path left out).
// FIRST (of an update): also the squared Frobenius norm of R less the path as the last sweep left it, by workgroup: the error after the
// update before this one
enum Pass { ITERATE, FIRST, FINAL };
template <int J, Pass PASS>
__global__ __launch_bounds__(256, PASS == FIRST && J == 2 ? 3 : 4) void rows_kernel(Problem<J> p, const double *b, double *a, double *a_sq, uint32_t *signs, double *err_sq, const Scalars *sc)
{
    if (PASS == FINAL ? !sc->done : sc->done) return;
    constexpr int N = PASS == FIRST ? J + 1 : J;
    __shared__ double red[4][ROWS], red_err[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = blockIdx.x * ROWS, r_last = p.out - 1;
    Rows<N> rows;
    fetch_rows<J, N>(p, r, r_last, rows);
    double dot[ROWS], sq = 0.0;
#pragma unroll
    for (int u = 0; u < ROWS; ++u) dot[u] = 0.0;
    auto safe = [&](int c) { return c < p.in ? c : 0; };       // in % 32 == 0: all four columns or none
    Piece<N> piece;
    fetch<J, N>(p, r, r_last, safe(4 * (int)threadIdx.x), piece);
#pragma unroll 1
    for (int c0 = 0; c0 < p.in; c0 += 1024) {
        const int c = c0 + 4 * (int)threadIdx.x, cs = safe(c);
        Columns<N> cols;
        double bv[4], v[ROWS][4];
        fetch_columns<J, N>(p, cs, cols);
        four(b, cs, bv);
        Piece<N> next;
        fetch<J, N>(p, r, r_last, safe(c + 1024), next);
        __builtin_amdgcn_sched_barrier(0);
        if (c >= p.in) bv[0] = bv[1] = bv[2] = bv[3] = 0.0;
        residuals<J, N>(p, piece, cols, rows, cs, v);
#pragma unroll
        for (int u = 0; u < ROWS; ++u) {
            if (PASS == FINAL) {
                // eight lanes hold the 32 columns of a word, four each
                uint32_t four = 0;
#pragma unroll
                for (int e = 0; e < 4; ++e) four |= !(v[u][e] >= 0.0) ? 1u << e : 0u;
                const uint32_t word = or_over_8(four << (4 * (lane & 7)));
                if ((lane & 7) == 0 && c < p.in && r + u < p.out) signs[(size_t)(r + u) * (p.in / 32) + (c >> 5)] = word;
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) dot[u] += fabs(v[u][e]) * bv[e];
        }
        if (PASS == FIRST) {
            subtract<N>(piece, cols, rows, J, cs, v);
#pragma unroll
            for (int u = 0; u < ROWS; ++u)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (r + u < p.out && c < p.in) sq += v[u][e] * v[u][e];
        }
        piece = next;
    }
#pragma unroll
    for (int u = 0; u < ROWS; ++u) {
        for (int m = 32; m > 0; m >>= 1) dot[u] += __shfl_xor(dot[u], m);
        if (lane == 0) red[wave][u] = dot[u];
    }
    if (PASS == FIRST) {
        for (int m = 32; m > 0; m >>= 1) sq += __shfl_xor(sq, m);
        if (lane == 0) red_err[wave] = sq;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    double s2 = 0.0;
#pragma unroll
    for (int u = 0; u < ROWS; ++u) {
        if (r + u >= p.out) break;
        const double s = ((red[0][u] + red[1][u]) + red[2][u]) + red[3][u];
        a[r + u] = s;
        s2 += s * s;
    }
    a_sq[blockIdx.x] = s2;
    if (PASS == FIRST) err_sq[blockIdx.x] = ((red_err[0] + red_err[1]) + red_err[2]) + red_err[3];
}

// partial[slice][c] = sum over the slice's rows of |R[r][c]| a[r]; a thread per four consecutive
// columns, the rows of the slice in order, ROWS at a time, the next ones in flight
template <int J>
__global__ __launch_bounds__(256, 4) void cols_kernel(Problem<J> p, const double *a, double *partial, int slice_rows, const Scalars *sc)
{
    if (sc->done) return;
    const int c = (blockIdx.x * 256 + threadIdx.x) * 4;
    const int r0 = blockIdx.y * slice_rows, r1 = min(p.out, r0 + slice_rows);
    if (c >= p.in) return;
    Columns<J> cols;
    fetch_columns<J, J>(p, c, cols);
    Piece<J> piece;
    fetch<J, J>(p, r0, r1 - 1, c, piece);
    double s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
    for (int r = r0; r < r1; r += ROWS) {
        Piece<J> next;
        fetch<J, J>(p, min(r + ROWS, r1 - 1), r1 - 1, c, next);
        Rows<J> rows;
        fetch_rows<J, J>(p, r, r1 - 1, rows);
        double a_r[ROWS], v[ROWS][4];
#pragma unroll
        for (int u = 0; u < ROWS; ++u) a_r[u] = r + u < r1 ? a[r + u] : 0.0;
        __builtin_amdgcn_sched_barrier(0);
        residuals<J, J>(p, piece, cols, rows, c, v);
#pragma unroll
        for (int u = 0; u < ROWS; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e] += fabs(v[u][e]) * a_r[u];
        piece = next;
    }
    double *dst = partial + (size_t)blockIdx.y * p.in + c;
    *reinterpret_cast<double2 *>(dst) = make_double2(s[0], s[1]);
    *reinterpret_cast<double2 *>(dst + 2) = make_double2(s[2], s[3]);
}

// Both passes of an iteration in one reading of W: a workgroup per compute unit takes a run of whole rows, one after the other, and
// keeps what it shares of the columns (the paths' h, the sums) in registers, four columns in each of CG groups of 2048 per
// thread, and b in LDS.  A row's R stays in registers from its dot product with b to its part of the column sums; the next row is
// on its way meanwhile (with two to four of them it was no faster).  The factor f of a column is taken out of it, R = f (rows W - g B h / f), and goes with b and with the column
// sums (a column without a factor has no h).  partial[workgroup][c] = sum over its rows of |R[r][c]| a[r], a_sq[workgroup]
// the sum of a[r]^2.
// LAST (after the iteration): a, the signs of R as rows_kernel<., FINAL> gives them (R in the order of its products, so the factors are
// in LDS and b in registers), and partial[workgroup] = the sum of (|R[r][c]| - a[r] b[c])^2, the error after this update: what the
// path leaves of R, while R is still there.  With that no pass after it has to find the error (a first pass by rows for it and one by columns
// took 68 us where an iteration is one of 38; the pass over all paths at the end 34).
// WALKS: the device goes through the updates by itself.  Before the rows, every workgroup does for itself what unit_kernel does: b from the sums
// of the iteration before, its change, the stopping rule, all from the same values in the same order, so all come to the same end and
// all take the same next step: an iteration, LAST, the first iteration of the next update (after a LAST; b is the all-ones vector then) or, after
// the last update, nothing.  The first workgroup writes down b and the scalars, where nobody reads them meanwhile.  So the host only has to
// ask for enough passes.  With a look after each update (27 us in which nothing runs, and launches for its start and end) ten updates of
// 4096 x 11008 took 2.70 ms and take 2.44 (without factors 2.60 and 2.22), 1024 x 2048 1.33 and 0.92, three paths 4096 x 8192 (nine updates)
// 2.17 and 1.94, one sweep of 4096 x 11008 0.57 and 0.54.  The columns' values are asked for before b is worked out, and the sums' factor is
// left to walk_sums_kernel: 2.46 to 2.44.
// Of a pass of 44 us over 4096 x 11008, 1.66 us are a row in each workgroup (6.9 TB/s) and 17 what it does once: 5 for a launch that has nothing to do,
// the rest the trip to memory for b and the sums, 48 divisions, the columns' values and the writing of its sums.  (A launch of its own for b, of one workgroup, took 7 us of an iteration's 50.)
// Bound: the reading of W; a row of 11008 columns costs a SIMD about 0.7 us of double precision and 0.3 us for the sum over the
// workgroup, and has 1.9 us in which 256 compute units read a row each.
constexpr int SUMS_COLS = 64, SUMS_RUNS = 8;       // (see slices_kernel)
constexpr int ONE_PASS_GROUPS = 256, ONE_PASS_THREADS = 512, GROUP_COLS = 4 * ONE_PASS_THREADS;
template <int N> struct RowPiece {
    float4 w;
    uint32_t bits[N + 1];
};
// Not for three paths of more than 8192 columns: LAST would spill 52 registers
// (169 us, where the pass by rows and a first iteration in two passes cost 66 more than an iteration; 4096 x 11008, three sweeps 4.10 and 3.42 ms)
constexpr bool walks(int J, int CG) { return J < 2 || CG < 6; }
// what a pass starts from and, where it walks, leaves for the next one
struct Step {
    const double *b, *sum, *sum_sq;
    double *b_new;
    const Scalars *sc;
    Scalars *sc_new;
    int n_sq, T_max;                   // values of sum_sq; sweeps
};
// p: WALKS: the first of the J + 1 paths, which lie one after the other; else the J paths to subtract
template <int J, int CG>
__global__ __launch_bounds__(ONE_PASS_THREADS, 2) void one_pass_kernel(Problem<J> p, uint32_t *packed, Step st, double *partial, double *a, double *a_sq)
{
    constexpr int WAVES = ONE_PASS_THREADS / 64;
    constexpr bool WALKS = walks(J, CG);
    extern __shared__ __attribute__((aligned(16))) double2 lds[];      // [CG][2][thread]: f b (LAST: f) of two columns, zero past the last column
    __shared__ double red[2][WAVES], red_group[WAVES];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, in = p.in, W32 = in / 32;
    const int r0 = (int)((long long)p.out * blockIdx.x / gridDim.x), r1 = (int)((long long)p.out * (blockIdx.x + 1) / gridDim.x);
    struct Row { RowPiece<J> piece[CG]; double factor, g[J + 1]; } row;
    const Scalars before = *st.sc;                             // (looked at when the first loads are on their way)
    // (buffer loads: columns past the last one read as zero, and one register holds the thread's place in every group.  A scalar offset
    // beside it is no part of the check, so only groups that the row fills have one; the last two, which it may not, are buffers of their own)
    auto buffer = [](const void *row, int bytes, int at) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(static_cast<const uint8_t *>(row)) + min(at, bytes), 0, max(bytes - at, 0), 0x00020000);
    };
    auto each_group = [&](const void *row, int bytes, int group_bytes, auto load) {
        const __amdgpu_buffer_rsrc_t filled = buffer(row, bytes, 0);
#pragma unroll
        for (int k = 0; k < CG - 2; ++k) load(k, filled, k * group_bytes);
#pragma unroll
        for (int k = CG - 2; k < CG; ++k) load(k, buffer(row, bytes, k * group_bytes), 0);
    };
    auto column = [&](int k) { return k * GROUP_COLS + 4 * tid; };
    auto safe = [&](int c) { return c < in ? c : 0; };          // in % 32 == 0: all four columns exist or none
    auto fetch_weights = [&](int r) {
        each_group(p.W + (size_t)r * in, in * 4, GROUP_COLS * 4, [&](int k, __amdgpu_buffer_rsrc_t rs, int at) {
            row.piece[k].w = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rs, tid * 16, at, 0));
        });
    };
    // WALKS: path j of those that the update subtracts is j or, from the one left out on, j + 1.  (Made scalars where they are used: with
    // pointers worked out at the start the compiler had a loop over the lanes around each load of a buffer, and a pass took 7 us more)
    struct Paths { int n[J + 1]; };
    auto paths_without = [](int left_out) {
        const int i = __builtin_amdgcn_readfirstlane(left_out);
        Paths to;
#pragma unroll
        for (int j = 0; j < J; ++j) to.n[j] = WALKS ? j + (j >= i) : 0;
        return to;
    };
    auto fetch_paths = [&](int r, const Paths &paths) {
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int from = WALKS ? 0 : j;
            const size_t line = (size_t)paths.n[j] * p.out + r;
            each_group(p.packed[from] + line * W32, W32 * 4, GROUP_COLS / 8, [&](int k, __amdgpu_buffer_rsrc_t rs, int at) {
                row.piece[k].bits[j] = __builtin_amdgcn_raw_buffer_load_b32(rs, tid / 8 * 4, at, 0);
            });
            row.g[j] = p.g[from][line];
        }
        row.factor = p.rows ? p.rows[r] : 1.0;                 // (a branch: what comes after it is asked for after the row before has been waited for)
    };
    // what the pass shares of the columns.  WALKS: on its way while b is worked out (three paths of 12288 columns have no registers for that:
    // 13 instead of 11 spill, 2048 x 11008 5 % slower)
    Columns<J> cols[CG];
    auto fetch_shared = [&](int k, const Paths &paths) {
        const int c = safe(column(k));
        cols[k].f[0] = cols[k].f[1] = cols[k].f[2] = cols[k].f[3] = 1.0;
        if (p.cols) four(p.cols, c, cols[k].f);
#pragma unroll
        for (int j = 0; j < J; ++j) four(WALKS ? p.h[0] + (size_t)paths.n[j] * in : p.h[j], c, cols[k].h[j]);
    };
    int left_out = 0;
    fetch_weights(min(r0, p.out - 1));
    if (!WALKS) fetch_paths(min(r0, p.out - 1), Paths{});
    double b[CG][4];
#pragma unroll
    for (int k = 0; k < CG; ++k) four(st.b, safe(column(k)), b[k]);
    bool done = before.done != 0;
    if (WALKS) {
        static_assert(CG * GROUP_COLS / SUMS_COLS <= ONE_PASS_THREADS, "a thread takes one of the squares");
        double sum[CG][4], sq = st.sum_sq[min(tid, st.n_sq - 1)];
#pragma unroll
        for (int k = 0; k < CG; ++k) four(st.sum, safe(column(k)), sum[k]);
        // which update, and the paths that it subtracts
        Scalars after = before;
        const bool fresh = __builtin_amdgcn_readfirstlane(before.done) != 0;
        int t = __builtin_amdgcn_readfirstlane(before.t), i = __builtin_amdgcn_readfirstlane(before.i);
        if (fresh && ++i > J) {
            i = 0;
            ++t;
        }
        if (t >= st.T_max) {
            after.done = WALKED;
            after.t = t;
            after.i = -1;
            if (blockIdx.x == 0 && tid == 0) *st.sc_new = after;
            return;
        }
        left_out = i;
        fetch_paths(min(r0, p.out - 1), paths_without(i));
#pragma unroll
        for (int k = 0; k < CG; ++k) fetch_shared(k, paths_without(i));
        if (fresh) {
            after = Scalars{0.0, 0.0, 0.0, 0, 0, t, i};
            done = false;
            const double one = 1.0 / sqrt((double)in);
#pragma unroll
            for (int k = 0; k < CG; ++k)
#pragma unroll
                for (int e = 0; e < 4; ++e) b[k][e] = one;
        } else if (before.na == 0.0) {                         // |R| b = 0: b stays
            done = true;
        } else {
            after.sigma = sqrt(group_sum(tid < st.n_sq ? sq : 0.0, red_group, WAVES));
            double change = 0.0;
#pragma unroll
            for (int k = 0; k < CG; ++k)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const double bn = sum[k][e] / after.sigma, d = bn - b[k][e];
                    change += column(k) < in ? d * d : 0.0;
                    b[k][e] = bn;
                }
            after.db = sqrt(group_sum(change, red_group, WAVES));
            after.iters += 1;
            done = (fabs(after.sigma - before.sigma) <= TOL_SIGMA * after.sigma && after.db <= TOL_B) || after.iters >= MAX_ITER;
        }
        done = __builtin_amdgcn_readfirstlane(done);           // (the same everywhere)
        after.done = done;
        if (blockIdx.x == 0) {
#pragma unroll
            for (int k = 0; k < CG; ++k)
                if (column(k) < in) {
                    *reinterpret_cast<double2 *>(st.b_new + column(k)) = make_double2(b[k][0], b[k][1]);
                    *reinterpret_cast<double2 *>(st.b_new + column(k) + 2) = make_double2(b[k][2], b[k][3]);
                }
            if (tid == 0) *st.sc_new = after;
        }
    } else if (done) {
        return;
    }
    double squares = 0.0;
    auto over_rows = [&](auto last) {
        constexpr bool LAST = decltype(last)::value;
        double h[CG][J + 1][4], sum[CG][4], error = 0.0;
        uint32_t *const signs = packed + (size_t)__builtin_amdgcn_readfirstlane(left_out) * p.out * W32;
        const Paths paths = paths_without(left_out);
#pragma unroll
        for (int k = 0; k < CG; ++k) {
            const bool there = column(k) < in;
            if (!WALKS) fetch_shared(k, Paths{});
            double kept[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                b[k][e] = there ? b[k][e] : 0.0;
                kept[e] = LAST ? (there ? cols[k].f[e] : 0.0) : b[k][e] * fabs(cols[k].f[e]);
#pragma unroll
                for (int j = 0; j < J; ++j) {
                    if (LAST) h[k][j][e] = there ? cols[k].h[j][e] : 0.0;
                    else h[k][j][e] = cols[k].f[e] != 0.0 ? cols[k].h[j][e] / cols[k].f[e] : 0.0;
                }
                sum[k][e] = 0.0;
            }
            lds[2 * k * ONE_PASS_THREADS + tid] = make_double2(kept[0], kept[1]);
            lds[(2 * k + 1) * ONE_PASS_THREADS + tid] = make_double2(kept[2], kept[3]);
        }
        // (a thread reads what it has written there)
#pragma unroll 1
        for (int r = r0; r < r1; ++r) {
            double v[CG][4];
#pragma unroll
            for (int k = 0; k < CG; ++k) {
                const float w[4] = {row.piece[k].w.x, row.piece[k].w.y, row.piece[k].w.z, row.piece[k].w.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) v[k][e] = row.factor * (double)w[e];
                if (LAST) {
                    const double2 low = lds[2 * k * ONE_PASS_THREADS + tid], high = lds[(2 * k + 1) * ONE_PASS_THREADS + tid];
                    v[k][0] *= low.x; v[k][1] *= low.y; v[k][2] *= high.x; v[k][3] *= high.y;
                }
#pragma unroll
                for (int j = 0; j < J; ++j) {
                    const uint32_t bits = row.piece[k].bits[j] >> (4 * (tid & 7));
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const unsigned long long flip = (unsigned long long)(bits << (31 - e) & 0x80000000u) << 32;
                        v[k][e] -= __builtin_bit_cast(double, __builtin_bit_cast(unsigned long long, row.g[j]) ^ flip) * h[k][j][e];
                    }
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            fetch_weights(min(r + 1, r1 - 1));
            fetch_paths(min(r + 1, r1 - 1), paths);
            __builtin_amdgcn_sched_barrier(0);
            double dot[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int k = 0; k < CG; ++k) {
                double2 low, high;
                if (LAST) {
                    low = make_double2(b[k][0], b[k][1]);
                    high = make_double2(b[k][2], b[k][3]);
                    // eight lanes hold the 32 columns of a word, four each
                    uint32_t four = 0;
#pragma unroll
                    for (int e = 0; e < 4; ++e) four |= !(v[k][e] >= 0.0) ? 1u << e : 0u;
                    const uint32_t word = or_over_8(four << (4 * (lane & 7)));
                    if ((lane & 7) == 0 && column(k) < in) signs[(size_t)r * W32 + (column(k) >> 5)] = word;
                } else {
                    low = lds[2 * k * ONE_PASS_THREADS + tid];
                    high = lds[(2 * k + 1) * ONE_PASS_THREADS + tid];
                }
                dot[0] += fabs(v[k][0]) * low.x;
                dot[1] += fabs(v[k][1]) * low.y;
                dot[2] += fabs(v[k][2]) * high.x;
                dot[3] += fabs(v[k][3]) * high.y;
            }
            const double d = over_wave((dot[0] + dot[1]) + (dot[2] + dot[3]));
            if (lane == 0) red[r & 1][wave] = d;
            __syncthreads();                                       // (the other half of `red` is written before anyone is a row further on)
            double ar = 0.0;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) ar += red[r & 1][w];
            squares += ar * ar;
            if (LAST && tid == 0) a[r] = ar;
#pragma unroll
            for (int k = 0; k < CG; ++k)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (LAST) {
                        const double left = fabs(v[k][e]) - ar * b[k][e];
                        error += left * left;
                    } else {
                        sum[k][e] += fabs(v[k][e]) * ar;
                    }
                }
        }
        if (LAST) {
            error = group_sum(error, red_group, WAVES);
            if (tid == 0) partial[blockIdx.x] = error;
        } else {
#pragma unroll
            for (int k = 0; k < CG; ++k) {
                const int c = column(k);
                if (c >= in) continue;
                double f[4] = {1.0, 1.0, 1.0, 1.0};
                if (!WALKS && p.cols) four(p.cols, c, f);        // (WALKS: by walk_sums_kernel, once for all workgroups)
                double *const to = partial + (size_t)blockIdx.x * in + c;
                *reinterpret_cast<double2 *>(to) = make_double2(sum[k][0] * fabs(f[0]), sum[k][1] * fabs(f[1]));
                *reinterpret_cast<double2 *>(to + 2) = make_double2(sum[k][2] * fabs(f[2]), sum[k][3] * fabs(f[3]));
            }
        }
    };
    if constexpr (WALKS) {
        if (done) over_rows(std::true_type{});
        else over_rows(std::false_type{});
    } else {
        over_rows(std::false_type{});
    }
    if (tid == 0) a_sq[blockIdx.x] = squares;
}
// groups of columns of the one-pass form, 0 where it is not taken.  Wider rows do not fit the registers; below 1024 rows (four per workgroup) the sums
// of 256 workgroups are as much to move as what a second pass reads, and rows of less than 2048 columns leave threads idle (time
// of the call over that with two passes: 4096 x 11008 0.70, 5504 x 8192 0.62, 11008 x 4096 0.68, three paths 4096 x 11008, where 12 registers spill,
// 0.86, 1024 x 11008 0.85, 1400 x 2048 0.75)
static int one_pass_groups(int out, int in)
{
    const int groups = (in + GROUP_COLS - 1) / GROUP_COLS;
    if (out < ONE_PASS_MIN_ROWS || in < ONE_PASS_MIN_COLS || groups > 6) return 0;
    return (groups + 1) / 2 * 2;
}
template <int J, int CG> static int launch_groups(const Problem<J> &p, uint32_t *packed, const Step &st, double *partial, double *a, double *a_sq, hipStream_t stream)
{
    constexpr int lds = CG * GROUP_COLS * (int)sizeof(double);
    static std::atomic<bool> allowed[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return RB_ERR_HIP;
    if (lds > 48 * 1024 && !allowed[dev].load()) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(one_pass_kernel<J, CG>), hipFuncAttributeMaxDynamicSharedMemorySize, lds) != hipSuccess) return RB_ERR_HIP;
        allowed[dev].store(true);
    }
    hipLaunchKernelGGL((one_pass_kernel<J, CG>), dim3(ONE_PASS_GROUPS), dim3(ONE_PASS_THREADS), lds, stream, p, packed, st, partial, a, a_sq);
    return RB_OK;
}
template <int J> static int launch_one_pass(int groups, const Problem<J> &p, uint32_t *packed, const Step &st, double *partial, double *a, double *a_sq, hipStream_t stream)
{
    if (groups == 2) return launch_groups<J, 2>(p, packed, st, partial, a, a_sq, stream);
    if (groups == 4) return launch_groups<J, 4>(p, packed, st, partial, a, a_sq, stream);
    return launch_groups<J, 6>(p, packed, st, partial, a, a_sq, stream);
}

// sum[c] = the slices of partial[.][c], in eight runs of consecutive ones, over the norm of a (every workgroup adds
// that up: squares of sums left at their length would leave fp64's range with W'^4), and the squares by workgroup
__global__ __launch_bounds__(SUMS_COLS * SUMS_RUNS) void slices_kernel(const double *partial, int n_slices, const double *a_sq, int n_a, int in, double *sum, double *sum_sq, Scalars *sc)
{
    const int done = sc->done;                                 // (looked at when the sums are there: no trip to memory before theirs)
    __shared__ double part[SUMS_RUNS][SUMS_COLS], red[SUMS_RUNS];
    const int x = threadIdx.x % SUMS_COLS, run = threadIdx.x / SUMS_COLS, c = blockIdx.x * SUMS_COLS + x, cs = min(c, in - 1);
    double s = 0.0, na = 0.0;
    for (int i = threadIdx.x; i < n_a; i += SUMS_COLS * SUMS_RUNS) na += a_sq[i];
#pragma unroll 8
    for (int k = n_slices * run / SUMS_RUNS; k < n_slices * (run + 1) / SUMS_RUNS; ++k) s += partial[(size_t)k * in + cs];
    if (done) return;
    part[run][x] = s;
    na = sqrt(group_sum(na, red, SUMS_RUNS));
    if (blockIdx.x == 0 && threadIdx.x == 0) sc->na = na;
    if (threadIdx.x >= SUMS_COLS) return;
    s = 0.0;
#pragma unroll
    for (int k = 0; k < SUMS_RUNS; ++k) s += part[k][x];
    s /= na;                                                   // (a zero norm: the next kernel does not look at the sums)
    if (c < in) sum[c] = s;
    double sq = c < in ? s * s : 0.0;
    for (int m = SUMS_COLS / 2; m > 0; m >>= 1) sq += __shfl_xor(sq, m);
    if (x == 0) sum_sq[blockIdx.x] = sq;
}

// g' and h' of path i as scales_kernel gives them, and the error after the update
struct Ends {
    const double *a, *b;
    double *g, *h, *err;               // [K][out], [K][in], [T_max][K] (or nullptr)
};
// What follows a pass of the walking form: the sums as slices_kernel makes them or, after a LAST, the path's scales as scales_kernel makes
// them.  (The first eight slices are asked for before it is known which: one trip to memory less)
__global__ __launch_bounds__(SUMS_COLS * SUMS_RUNS) void walk_sums_kernel(const double *partial, const double *a_sq, const double *cols, int K, int out, int in, double *sum, double *sum_sq, Ends to, Scalars *sc)
{
    constexpr int THREADS = SUMS_COLS * SUMS_RUNS, OF_RUN = ONE_PASS_GROUPS / SUMS_RUNS, FIRST = 8;
    static_assert(ONE_PASS_GROUPS <= THREADS && OF_RUN % FIRST == 0, "a thread takes one square; whole batches of slices");
    const int done = sc->done, t = sc->t, i = sc->i;
    __shared__ double part[SUMS_RUNS][SUMS_COLS], red[SUMS_RUNS];
    const int tid = threadIdx.x, x = tid % SUMS_COLS, run = tid / SUMS_COLS, c = blockIdx.x * SUMS_COLS + x;
    const double *from = partial + (size_t)(OF_RUN * run) * in + min(c, in - 1);
    const double factor = cols ? fabs(cols[min(c, in - 1)]) : 1.0;
    double na = tid < ONE_PASS_GROUPS ? a_sq[tid] : 0.0, held[FIRST];
#pragma unroll
    for (int k = 0; k < FIRST; ++k) held[k] = from[(size_t)k * in];
    if (done == WALKED) return;
    if (done) {
        const double sigma = sqrt(group_sum(na, red, SUMS_RUNS)), root = sqrt(sigma);
        for (int n = blockIdx.x * THREADS + tid; n < max(out, in); n += gridDim.x * THREADS) {
            if (n < out) to.g[(size_t)i * out + n] = sigma > 0.0 ? root * (to.a[n] / sigma) : 0.0;
            if (n < in) to.h[(size_t)i * in + n] = root * to.b[n];
        }
        if (to.err && blockIdx.x == 0) {
            const double e2 = group_sum(tid < ONE_PASS_GROUPS ? partial[tid] : 0.0, red, SUMS_RUNS);
            if (tid == 0) to.err[(size_t)t * K + i] = sqrt(e2);
        }
        return;
    }
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < FIRST; ++k) s += held[k];
#pragma unroll
    for (int k = FIRST; k < OF_RUN; ++k) s += from[(size_t)k * in];
    part[run][x] = s;
    na = sqrt(group_sum(na, red, SUMS_RUNS));
    if (blockIdx.x == 0 && tid == 0) sc->na = na;
    if (tid >= SUMS_COLS) return;
    s = 0.0;
#pragma unroll
    for (int k = 0; k < SUMS_RUNS; ++k) s += part[k][x];
    s = s * factor / na;                                                   // (a zero norm: the next pass does not look at the sums)
    if (c < in) sum[c] = s;
    double sq = c < in ? s * s : 0.0;
    for (int m = SUMS_COLS / 2; m > 0; m >>= 1) sq += __shfl_xor(sq, m);
    if (x == 0) sum_sq[blockIdx.x] = sq;
}
// as after a LAST: the first pass begins the first update
__global__ void walk_start_kernel(Scalars *sc) { *sc = Scalars{0.0, 0.0, 0.0, 1, 0, 0, -1}; }

constexpr int UNIT_HELD = 12;           // columns of a thread that the next kernel asks for at its start
// b_new = sum / its norm, the change of b, the stopping rule  (one workgroup)
__global__ __launch_bounds__(1024) void unit_kernel(double *b, const double *sum, const double *sum_sq, int in, Scalars *sc)
{
    if (sc->done) return;
    __shared__ double red[16];
    // (the first UNIT_HELD x 1024 columns are asked for before the norm is known: one trip to memory instead of two, 7.5 -> 6.6 us)
    double held_sum[UNIT_HELD], held_b[UNIT_HELD];
#pragma unroll
    for (int i = 0; i < UNIT_HELD; ++i) {
        held_sum[i] = held_b[i] = 0.0;
        if (1024 * i >= in) continue;
        const int c = min((int)threadIdx.x + 1024 * i, in - 1);
        held_sum[i] = sum[c];
        held_b[i] = b[c];
    }
    double sigma = 0.0;
    for (int i = threadIdx.x; i < (in + SUMS_COLS - 1) / SUMS_COLS; i += 1024) sigma += sum_sq[i];
    sigma = sqrt(group_sum(sigma, red, 16));
    if (sc->na == 0.0) {                                       // |R| b = 0: b stays
        if (threadIdx.x == 0) sc->done = 1;
        return;
    }
    double db = 0.0;
    auto update = [&](int c, double s, double old) {
        const double bn = s / sigma, d = bn - old;
        db += d * d;
        b[c] = bn;
    };
#pragma unroll
    for (int i = 0; i < UNIT_HELD; ++i)
        if ((int)threadIdx.x + 1024 * i < in) update(threadIdx.x + 1024 * i, held_sum[i], held_b[i]);
    for (int c = threadIdx.x + 1024 * UNIT_HELD; c < in; c += 1024) update(c, sum[c], b[c]);
    db = sqrt(group_sum(db, red, 16));
    if (threadIdx.x == 0) {
        const bool done = fabs(sigma - sc->sigma) <= TOL_SIGMA * sigma && db <= TOL_B;
        sc->sigma = sigma;
        sc->db = db;
        sc->iters += 1;
        if (done || sc->iters >= MAX_ITER) sc->done = 1;
    }
}

// after the final a = |R| b: g' = sqrt(sigma) a / sigma, h' = sqrt(sigma) b with sigma = ||a||
__global__ __launch_bounds__(256) void scales_kernel(const double *a, const double *b, const double *a_sq, int n_a, double *g_i,
                                                     double *h_i, int out, int in, const Scalars *sc)
{
    if (!sc->done) return;
    __shared__ double red[4];
    double a2 = 0.0;
    for (int i = threadIdx.x; i < n_a; i += 256) a2 += a_sq[i];
    a2 = group_sum(a2, red, 4);
    const double sigma = sqrt(a2), root = sqrt(sigma);
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < out) g_i[i] = sigma > 0.0 ? root * (a[i] / sigma) : 0.0;
    if (i < in) h_i[i] = root * b[i];
}

// squared Frobenius norm of W' - sum_j What_j over all J paths (the last update: nothing follows that could find it on the
// way), ROWS rows per workgroup as above, then one workgroup adds them up
template <int J>
__global__ __launch_bounds__(256, 4) void err_rows_kernel(Problem<J> p, double *rows_sq)
{
    __shared__ double red[4];
    const int r = blockIdx.x * ROWS, r_last = p.out - 1;
    Rows<J> rows;
    fetch_rows<J, J>(p, r, r_last, rows);
    double sq = 0.0;
    for (int c = 4 * (int)threadIdx.x; c < p.in; c += 1024) {
        double v[ROWS][4];
        Columns<J> cols;
        Piece<J> piece;
        fetch_columns<J, J>(p, c, cols);
        fetch<J, J>(p, r, r_last, c, piece);
        residuals<J, J>(p, piece, cols, rows, c, v);
#pragma unroll
        for (int u = 0; u < ROWS; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (r + u < p.out) sq += v[u][e] * v[u][e];
    }
    sq = group_sum(sq, red, 4);
    if (threadIdx.x == 0) rows_sq[blockIdx.x] = sq;
}
__global__ __launch_bounds__(1024) void err_sum_kernel(const double *rows_sq, int n, double *err)
{
    __shared__ double red[1024];
    double s = 0.0;
    for (int i = threadIdx.x; i < n; i += 1024) s += rows_sq[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = 512; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *err = sqrt(red[0]);
}

__global__ __launch_bounds__(256) void clear_kernel(double *v, size_t n, uint32_t *w, size_t nw)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) v[i] = 0.0;
    if (i < nw) w[i] = 0u;
}

// step 3: back to the original domain
__global__ __launch_bounds__(256) void unscale_kernel(double *g, double *h, const double *rows, const double *cols, int K, int out,
                                                      int in)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    for (int k = 0; k < K; ++k) {
        if (rows && i < out) g[(size_t)k * out + i] /= rows[i];
        if (cols && i < in) h[(size_t)k * in + i] /= cols[i];
    }
}

struct Layout {
    size_t scalars, a, a_sq, b, sum, sum_sq, partial, total;
};
// the slices come last; `rows` of them each, or the workgroups of the one-pass form and a second b
static Layout make_layout(int out, int in, int rows, bool one_pass)
{
    auto up = [](size_t v) { return (v + 255) / 256 * 256; };
    const size_t slices = std::max<size_t>((size_t)(out + rows - 1) / rows, one_pass ? ONE_PASS_GROUPS + 1 : 0), groups = (size_t)(out + ROWS - 1) / ROWS;
    Layout L;
    size_t o = 0;
    L.scalars = o; o += up(2 * sizeof(Scalars));
    L.a = o; o += up(sizeof(double) * out);
    L.a_sq = o; o += up(sizeof(double) * groups);
    L.b = o; o += up(sizeof(double) * in);
    L.sum = o; o += up(sizeof(double) * in);
    L.sum_sq = o; o += up(sizeof(double) * ((in + SUMS_COLS - 1) / SUMS_COLS));
    L.partial = o; o += up(sizeof(double) * slices * in);
    L.total = o;
    return L;
}

struct Buffers {
    Scalars *sc;
    double *a, *a_sq, *b, *sum, *sum_sq, *partial;
};

// All updates by one_pass_kernel where it walks.  The host asks for a first sweep's passes and looks how far they came; then for as many as
// passes_to_ask says, and looks again.
template <int K>
static int walk(const Problem<K - 1> &p, uint32_t *packed, double *g, double *h, double *err, int T_max, int groups, const Buffers &ws, hipStream_t stream)
{
    const int in = p.in, n_sq = (in + SUMS_COLS - 1) / SUMS_COLS;
    double *const bs[2] = {ws.b, ws.partial + (size_t)ONE_PASS_GROUPS * in};
    hipLaunchKernelGGL(walk_start_kernel, dim3(1), dim3(1), 0, stream, ws.sc);
    double passes = 0.0;
    for (int now = 0, n = K * (FIRST_LOOK + 1);;) {
        for (int k = 0; k < n; ++k, now ^= 1) {
            const Step st{bs[now], ws.sum, ws.sum_sq, bs[now ^ 1], ws.sc + now, ws.sc + (now ^ 1), n_sq, T_max};
            const int rc = launch_one_pass(groups, p, packed, st, ws.partial, ws.a, ws.a_sq, stream);
            if (rc != RB_OK) return rc;
            hipLaunchKernelGGL(walk_sums_kernel, dim3(n_sq), dim3(SUMS_COLS * SUMS_RUNS), 0, stream, ws.partial, ws.a_sq, p.cols, K, p.out, in, ws.sum, ws.sum_sq,
                               Ends{ws.a, bs[now ^ 1], g, h, err}, ws.sc + (now ^ 1));
        }
        Scalars host;
        if (hipMemcpyAsync(&host, ws.sc + now, sizeof(host), hipMemcpyDeviceToHost, stream) != hipSuccess || hipStreamSynchronize(stream) != hipSuccess)
            return RB_ERR_HIP;
        passes += n;
        const double under_way = host.done ? 0.0 : host.iters + 1.0, finished = (double)K * host.t + host.i + (host.done ? 1.0 : 0.0), left = (double)K * T_max - finished;
        if (host.done == WALKED || left <= 0.0) return RB_OK;
        n = passes_to_ask(passes, under_way, finished, left);
    }
}

template <int K>
static int derive(const float *W, const double *row_factors, const double *col_factors, int out, int in, int T_max, double *g, double *h,
                  uint32_t *packed, double *err, const Buffers &ws, int slice_rows, bool room, hipStream_t stream)
{
    const int one_pass = room ? one_pass_groups(out, in) : 0;
    const size_t words = (size_t)out * (in / 32);
    if (one_pass && walks(K - 1, one_pass)) {
        Problem<K - 1> all{W, row_factors, col_factors, {}, {}, {}, out, in};
        for (int j = 0; j < K; ++j) {
            all.packed[j] = packed + j * words;
            all.g[j] = g + (size_t)j * out;
            all.h[j] = h + (size_t)j * in;
        }
        return walk<K>(all, packed, g, h, err, T_max, one_pass, ws, stream);
    }
    const int n_slices = (out + slice_rows - 1) / slice_rows, n_a = (out + ROWS - 1) / ROWS;
    const dim3 by_rows((unsigned)n_a), by_cols((in + 1023) / 1024, n_slices), wg(256);
    int look = FIRST_LOOK;                         // iterations enqueued before the host looks: as many as the last update took
    for (int t = 0; t < T_max; ++t) {
        for (int i = 0; i < K; ++i) {
            // the paths but i, and i itself as the last sweep left it (nothing, in the first) at the end
            Problem<K - 1> p{W, row_factors, col_factors, {}, {}, {}, out, in};
            for (int j = 0, n = 0; j < K; ++j) {
                const int at = j == i ? K - 1 : n++;
                p.packed[at] = packed + j * words;
                p.g[at] = g + (size_t)j * out;
                p.h[at] = h + (size_t)j * in;
            }
            uint32_t *const signs = packed + i * words;
            const bool err_before = err && t * K + i > 0;
            hipLaunchKernelGGL(start_kernel, dim3((in + 255) / 256), wg, 0, stream, ws.b, in, ws.sc);
            double *const err_here = err ? err + (size_t)t * K + i : nullptr;
            Scalars host;
            for (int it = 1;; ++it) {
                const bool one = one_pass && (it > 1 || !err_before);
                if (one) {
                    const int rc = launch_one_pass(one_pass, p, packed, Step{ws.b, nullptr, nullptr, nullptr, ws.sc, nullptr, 0, 0}, ws.partial, ws.a, ws.a_sq, stream);
                    if (rc != RB_OK) return rc;
                } else {
                    if (it == 1 && err_before) {
                        // (`partial` has room: out / 4 sums where the column pass has in >= 32 for every 32 rows, or 64 with the smaller workspace)
                        hipLaunchKernelGGL((rows_kernel<K - 1, FIRST>), by_rows, wg, 0, stream, p, ws.b, ws.a, ws.a_sq, signs, ws.partial, ws.sc);
                        hipLaunchKernelGGL(err_sum_kernel, dim3(1), dim3(1024), 0, stream, ws.partial, n_a, err_here - 1);
                    } else {
                        hipLaunchKernelGGL((rows_kernel<K - 1, ITERATE>), by_rows, wg, 0, stream, p, ws.b, ws.a, ws.a_sq, signs, ws.partial, ws.sc);
                    }
                    hipLaunchKernelGGL((cols_kernel<K - 1>), by_cols, wg, 0, stream, p, ws.a, ws.partial, slice_rows, ws.sc);
                }
                hipLaunchKernelGGL(slices_kernel, dim3((in + SUMS_COLS - 1) / SUMS_COLS), dim3(SUMS_COLS * SUMS_RUNS), 0, stream, ws.partial, one ? ONE_PASS_GROUPS : n_slices, ws.a_sq,
                                   one ? ONE_PASS_GROUPS : n_a, in, ws.sum, ws.sum_sq, ws.sc);
                hipLaunchKernelGGL(unit_kernel, dim3(1), dim3(1024), 0, stream, ws.b, ws.sum, ws.sum_sq, in, ws.sc);
                if (it < look) continue;
                // |R| b and the signs for the converged b, the path's new scales: nothing happens unless the iteration has finished
                hipLaunchKernelGGL((rows_kernel<K - 1, FINAL>), by_rows, wg, 0, stream, p, ws.b, ws.a, ws.a_sq, signs, ws.partial, ws.sc);
                hipLaunchKernelGGL(scales_kernel, dim3((std::max(out, in) + 255) / 256), wg, 0, stream, ws.a, ws.b, ws.a_sq, n_a,
                                   g + (size_t)i * out, h + (size_t)i * in, out, in, ws.sc);
                if (hipMemcpyAsync(&host, ws.sc, sizeof(host), hipMemcpyDeviceToHost, stream) != hipSuccess ||
                    hipStreamSynchronize(stream) != hipSuccess)
                    return RB_ERR_HIP;
                if (host.done) break;
            }
            look = std::max(1, host.iters);
        }
    }
    if (err) {
        Problem<K> p{W, row_factors, col_factors, {}, {}, {}, out, in};
        for (int j = 0; j < K; ++j) {
            p.packed[j] = packed + j * words;
            p.g[j] = g + (size_t)j * out;
            p.h[j] = h + (size_t)j * in;
        }
        hipLaunchKernelGGL((err_rows_kernel<K>), by_rows, wg, 0, stream, p, ws.a);               // (a has been used up)
        hipLaunchKernelGGL(err_sum_kernel, dim3(1), dim3(1024), 0, stream, ws.a, n_a, err + (size_t)T_max * K - 1);
    }
    return RB_OK;
}

}  // namespace derive
}  // namespace rb

extern "C" size_t rb_derive_workspace_bytes(int out, int in)
{
    if (out < 1 || in < 32 || in % 32 != 0) return 0;
    return rb::derive::make_layout(out, in, rb::derive::ROW_SLICE, rb::derive::one_pass_groups(out, in) != 0).total;
}

extern "C" int rb_derive_iterative(const float *W, const double *row_factors, const double *col_factors, int K, int T_max,
                                   int out, int in, uint32_t *packed, double *g, double *h, double *err, void *workspace,
                                   size_t workspace_bytes, void *stream_)
{
    using namespace rb::derive;
    if (!W || !packed || !g || !h) return RB_ERR_NULL;
    if (K < 1 || K > RB_MAX_K || T_max < 1 || out < 1 || in < 32 || in % 32 != 0) return RB_ERR_SHAPE;
    if ((uintptr_t)packed & 3) return RB_ERR_ALIGN;
    if (((uintptr_t)g | (uintptr_t)row_factors | (uintptr_t)err) & 7) return RB_ERR_ALIGN;
    if (((uintptr_t)W | (uintptr_t)h | (uintptr_t)col_factors) & 15) return RB_ERR_ALIGN;      // read 16 bytes at a time
    // a smaller workspace (slices of twice the rows) does as well; more slices than the second dimension of a grid
    // may have: the same
    const bool short_slices = workspace_bytes >= make_layout(out, in, ROW_SLICE, false).total && out <= MAX_SLICES * ROW_SLICE;
    const int slice_rows = short_slices ? ROW_SLICE : 2 * ROW_SLICE;
    // (with less room than is asked for now: two passes)
    const bool room = one_pass_groups(out, in) && workspace_bytes >= make_layout(out, in, slice_rows, true).total;
    const Layout lay = make_layout(out, in, slice_rows, room);
    if (!workspace || workspace_bytes < lay.total) return RB_ERR_WORKSPACE;
    if ((uintptr_t)workspace & 15) return RB_ERR_ALIGN;
    hipStream_t stream = static_cast<hipStream_t>(stream_);
    uint8_t *ws = static_cast<uint8_t *>(workspace);
    auto at = [&](size_t offset) { return reinterpret_cast<double *>(ws + offset); };
    const Buffers buf{reinterpret_cast<Scalars *>(ws + lay.scalars), at(lay.a), at(lay.a_sq), at(lay.b), at(lay.sum),
                      at(lay.sum_sq), at(lay.partial)};
    const int W32 = in / 32;

    // What_i^(0) = 0: zero scales (and all-plus signs, which the zero scales make irrelevant)
    const size_t nv = (size_t)K * std::max(out, in), nw = (size_t)K * out * W32;
    hipLaunchKernelGGL(clear_kernel, dim3((unsigned)((std::max(nv, nw) + 255) / 256)), dim3(256), 0, stream, g,
                       (size_t)K * out, packed, nw);
    hipLaunchKernelGGL(clear_kernel, dim3((unsigned)(((size_t)K * in + 255) / 256)), dim3(256), 0, stream, h, (size_t)K * in,
                       static_cast<uint32_t *>(nullptr), (size_t)0);
    auto run = [&](auto derive_k) { return derive_k(W, row_factors, col_factors, out, in, T_max, g, h, packed, err, buf, slice_rows, room, stream); };
    const int rc = K == 1 ? run(derive<1>) : K == 2 ? run(derive<2>) : run(derive<3>);
    if (rc != RB_OK) return rc;
    if (row_factors || col_factors)
        hipLaunchKernelGGL(unscale_kernel, dim3((std::max(out, in) + 255) / 256), dim3(256), 0, stream, g, h, row_factors,
                           col_factors, K, out, in);
    if (hipGetLastError() != hipSuccess) return RB_ERR_HIP;
    return hipStreamSynchronize(stream) == hipSuccess ? RB_OK : RB_ERR_HIP;
}
