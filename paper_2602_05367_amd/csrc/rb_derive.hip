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
// all-ones vector (the matrix is non-negative): two passes per iteration, a = |R| b by rows (four rows
// per workgroup) and c = |R|^T a by columns (slices of rows, partial sums added in slice order); in both a lane takes
// four consecutive columns, one 16-byte load of W.  a is left at its length and its norm taken
// out of c: with b of length 1, sigma = ||c|| and the next b is c / ||c||.  After the last iteration one more pass by rows gives the last |R| b and the
// signs of R_i.  The error after an update, term by term (as ||R_i||^2 - sigma^2 it would come out of the same pass, but with
// a digit less: 3.6e-15 off where the terms are 1e-16), is found by the first pass of the next update on the way: its R less the
// path that it leaves out.  Every sum has a fixed order.  The
// iteration's stopping rule is evaluated on the device; the host reads one flag per update when it expects the
// iteration to have finished, so the call synchronises.
//
// Measured, 4096 x 11008, two paths, five sweeps (ten updates of four iterations): 3.9 ms (5.1 with the path left out found at
// run time, whose branches waited for every sign word by itself, nothing of the next step in flight, and passes of their own for the
// errors): a row pass 31 us (37 before), a column pass 31 us (47), the sums and the normalisation 13 us.  180 MB of W in
// 31 us are 5.8 TB/s, what a plain read of as much out of the memory-side cache reaches (6.0).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "rabit.h"
#include "rb_device.h"
#include "rb_internal.h"

namespace rb {
namespace derive {

constexpr int ROW_SLICE = 32;          // rows one workgroup of the column pass walks (twice that where the workspace is the smaller)
constexpr int MAX_SLICES = 65535;
constexpr int ROWS = 4;                // rows one workgroup of the row pass takes
constexpr int FIRST_LOOK = 4;          // power iterations before the first look at the flag
constexpr int MAX_ITER = 200;
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
    int done;           // the stopping rule held (or the matrix is zero)
    int iters;
};

// sum over a workgroup of `waves` wavefronts in a fixed order, in every thread; red has a slot per wavefront
__device__ __forceinline__ double group_sum(double v, double *red, int waves)
{
    for (int m = 32; m > 0; m >>= 1) v += __shfl_xor(v, m);
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

// sum[c] = the slices of partial[.][c], in eight runs of consecutive ones, over the norm of a (every workgroup adds
// that up: squares of sums left at their length would leave fp64's range with W'^4), and the squares by workgroup
constexpr int SUMS_COLS = 64, SUMS_RUNS = 8;
__global__ __launch_bounds__(SUMS_COLS * SUMS_RUNS) void slices_kernel(const double *partial, int n_slices, const double *a_sq, int n_a, int in, double *sum, double *sum_sq, Scalars *sc)
{
    if (sc->done) return;
    __shared__ double part[SUMS_RUNS][SUMS_COLS], red[SUMS_RUNS];
    const int x = threadIdx.x % SUMS_COLS, run = threadIdx.x / SUMS_COLS, c = blockIdx.x * SUMS_COLS + x, cs = min(c, in - 1);
    double s = 0.0, na = 0.0;
    for (int i = threadIdx.x; i < n_a; i += SUMS_COLS * SUMS_RUNS) na += a_sq[i];
#pragma unroll 8
    for (int k = n_slices * run / SUMS_RUNS; k < n_slices * (run + 1) / SUMS_RUNS; ++k) s += partial[(size_t)k * in + cs];
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

// b_new = sum / its norm, the change of b, the stopping rule  (one workgroup)
__global__ __launch_bounds__(1024) void unit_kernel(double *b, const double *sum, const double *sum_sq, int in, Scalars *sc)
{
    if (sc->done) return;
    __shared__ double red[16];
    double sigma = 0.0;
    for (int i = threadIdx.x; i < (in + SUMS_COLS - 1) / SUMS_COLS; i += 1024) sigma += sum_sq[i];
    sigma = sqrt(group_sum(sigma, red, 16));
    if (sc->na == 0.0) {                                       // |R| b = 0: b stays
        if (threadIdx.x == 0) sc->done = 1;
        return;
    }
    double db = 0.0;
#pragma unroll 4
    for (int c = threadIdx.x; c < in; c += 1024) {
        const double bn = sum[c] / sigma, d = bn - b[c];
        db += d * d;
        b[c] = bn;
    }
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
// the slices come last; `rows` of them each
static Layout make_layout(int out, int in, int rows)
{
    auto up = [](size_t v) { return (v + 255) / 256 * 256; };
    const size_t slices = (size_t)(out + rows - 1) / rows, groups = (size_t)(out + ROWS - 1) / ROWS;
    Layout L;
    size_t o = 0;
    L.scalars = o; o += up(sizeof(Scalars));
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

template <int K>
static int derive(const float *W, const double *row_factors, const double *col_factors, int out, int in, int T_max, double *g, double *h,
                  uint32_t *packed, double *err, const Buffers &ws, int slice_rows, hipStream_t stream)
{
    const int n_slices = (out + slice_rows - 1) / slice_rows, n_a = (out + ROWS - 1) / ROWS;
    const size_t words = (size_t)out * (in / 32);
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
            Scalars host;
            for (int it = 1;; ++it) {
                if (it == 1 && err_before) {
                    // (`partial` has room: out / 4 sums where the column pass has in >= 32 for every 32 rows, or 64 with the smaller workspace)
                    hipLaunchKernelGGL((rows_kernel<K - 1, FIRST>), by_rows, wg, 0, stream, p, ws.b, ws.a, ws.a_sq, signs, ws.partial, ws.sc);
                    hipLaunchKernelGGL(err_sum_kernel, dim3(1), dim3(1024), 0, stream, ws.partial, n_a, err + (size_t)t * K + i - 1);
                } else {
                    hipLaunchKernelGGL((rows_kernel<K - 1, ITERATE>), by_rows, wg, 0, stream, p, ws.b, ws.a, ws.a_sq, signs, ws.partial, ws.sc);
                }
                hipLaunchKernelGGL((cols_kernel<K - 1>), by_cols, wg, 0, stream, p, ws.a, ws.partial, slice_rows, ws.sc);
                hipLaunchKernelGGL(slices_kernel, dim3((in + SUMS_COLS - 1) / SUMS_COLS), dim3(SUMS_COLS * SUMS_RUNS), 0, stream, ws.partial, n_slices, ws.a_sq, n_a, in, ws.sum, ws.sum_sq, ws.sc);
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
    return rb::derive::make_layout(out, in, rb::derive::ROW_SLICE).total;
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
    const bool short_slices = workspace_bytes >= make_layout(out, in, ROW_SLICE).total && out <= MAX_SLICES * ROW_SLICE;
    const int slice_rows = short_slices ? ROW_SLICE : 2 * ROW_SLICE;
    const Layout lay = make_layout(out, in, slice_rows);
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
    auto run = [&](auto derive_k) { return derive_k(W, row_factors, col_factors, out, in, T_max, g, h, packed, err, buf, slice_rows, stream); };
    const int rc = K == 1 ? run(derive<1>) : K == 2 ? run(derive<2>) : run(derive<3>);
    if (rc != RB_OK) return rc;
    if (row_factors || col_factors)
        hipLaunchKernelGGL(unscale_kernel, dim3((std::max(out, in) + 255) / 256), dim3(256), 0, stream, g, h, row_factors,
                           col_factors, K, out, in);
    if (hipGetLastError() != hipSuccess) return RB_ERR_HIP;
    return hipStreamSynchronize(stream) == hipSuccess ? RB_OK : RB_ERR_HIP;
}
