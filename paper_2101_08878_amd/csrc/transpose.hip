// Sum of a matrix and its transpose: y = x + x^T, float64 (arXiv 2101.08878,
// Section V-B, "Sum of cuPy Array and its Transpose": the benchmark adds a
// chunked cuPy array to its transpose).
//
// HBM-bound: every element of x is read once and every element of y written
// once.  The matrix is cut into square tiles; a workgroup takes one tile pair
// (I, J) with I <= J and writes y[I, J] = x[I, J] + x[J, I]^T and y[J, I] =
// x[J, I] + x[I, J]^T.  Tiles are transposed through LDS (rows padded by one
// element, so that reading a column touches consecutive banks).  Each element
// is one IEEE-754 addition, the same on any device.
#include "mdx.h"
#include "mdx_internal.hpp"

namespace mdx {
namespace {

// Small, odd and unaligned matrices: 32 x 32 tiles, 256 threads, both tiles of
// the pair in LDS before either is written (so y may be x).  17 KB of LDS, so
// many workgroups share a CU and keep loads in flight.
constexpr int kTT = 32;                    // tile edge
constexpr int kTThreads = 256;
constexpr int kTRows = kTThreads / kTT;    // rows a workgroup moves per step
static_assert(kTT % kTRows == 0, "tile rows split evenly over the steps");

// Tile pair of workgroup p: pairs are numbered row by row over I <= J, so
// row I starts at I T - I (I - 1) / 2.
__device__ __forceinline__ void pair_of(int64_t p, int64_t T, int64_t &I, int64_t &J)
{
    const double b = 2.0 * (double)T + 1.0;
    int64_t i = (int64_t)((b - sqrt(b * b - 8.0 * (double)p)) * 0.5);
    i = i < 0 ? 0 : (i >= T ? T - 1 : i);
    auto start = [T](int64_t r) { return r * T - r * (r - 1) / 2; };
    while (i > 0 && start(i) > p)
        --i;
    while (i + 1 < T && start(i + 1) <= p)
        ++i;
    I = i;
    J = i + (p - start(i));
}

__global__ __launch_bounds__(kTThreads) void transpose_sum_tiles(const double *x, double *y, int64_t n,
                                                             int64_t T)
{
    __shared__ double a[kTT][kTT + 1], b[kTT][kTT + 1];
    int64_t I, J;
    pair_of(blockIdx.x, T, I, J);
    const int c = threadIdx.x % kTT, r0 = threadIdx.x / kTT;
    const int64_t i0 = I * kTT, j0 = J * kTT;
    const bool diag = I == J;
#pragma unroll
    for (int k = 0; k < kTT / kTRows; ++k) {
        const int r = r0 + k * kTRows;
        const int64_t ra = i0 + r, ca = j0 + c;  // x[I, J]
        if (ra < n && ca < n)
            a[r][c] = x[ra * n + ca];
        const int64_t rb = j0 + r, cb = i0 + c;  // x[J, I]
        if (!diag && rb < n && cb < n)
            b[r][c] = x[rb * n + cb];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kTT / kTRows; ++k) {
        const int r = r0 + k * kTRows;
        const int64_t ra = i0 + r, ca = j0 + c;
        if (ra < n && ca < n)
            y[ra * n + ca] = a[r][c] + (diag ? a[c][r] : b[c][r]);
        const int64_t rb = j0 + r, cb = i0 + c;
        if (!diag && rb < n && cb < n)
            y[rb * n + cb] = b[r][c] + a[c][r];
    }
}

// Large matrices: 128 x 128 tiles, 1024 threads, so that a tile's row is 1 KB
// of the matrix in one piece (32 x 32 tiles: 256 bytes, which the memory
// serves at 4.9 TB/s; 64 x 64: 5.2; 128 x 128: 5.4; float64, 16384 x 16384: 863,
// 826 and 793 us).  A thread holds its elements of both tiles in registers;
// one tile at a time passes through the 132 KB of LDS.  An element of y is
// written by the thread that read it from x, so y may be x.  Stores stream past
// the caches; loads do when the matrix is well beyond the 256 MB Infinity
// Cache (5120 x 5120: 64 us, with streaming loads 81; 16384 x 16384: 806 and
// 793).
constexpr int kBT = 128;
constexpr int kBThreads = 1024;
constexpr int kBCols = kBT / 2;             // threads per row, two elements each
constexpr int kBRows = kBThreads / kBCols;  // rows a workgroup moves per step
constexpr int kBSteps = kBT / kBRows;
constexpr int64_t kBigPairs = 768;                 // three workgroups for every CU
constexpr int64_t kStreamBytes = (int64_t)384 << 20;

typedef double f64x2 __attribute__((ext_vector_type(2)));

template <bool STREAM>
__global__ __launch_bounds__(kBThreads) void transpose_sum_big(const double *x, double *y,
                                                               int64_t n, int64_t T)
{
    __shared__ double t[kBT][kBT + 1];
    int64_t I, J;
    pair_of(blockIdx.x, T, I, J);
    const int c = (threadIdx.x % kBCols) * 2, r0 = threadIdx.x / kBCols;
    const int64_t i0 = I * kBT, j0 = J * kBT;
    // rows r0 + k kBRows, columns c and c + 1 of the tile at (row, col); n is
    // even, so the two columns lie in the matrix or both outside
    auto load = [&](int64_t row, int64_t col, f64x2 *v) {
#pragma unroll
        for (int k = 0; k < kBSteps; ++k) {
            const int64_t r = row + r0 + k * kBRows;
            v[k] = f64x2(0);
            if (r < n && col + c < n) {
                const f64x2 *p = (const f64x2 *)(x + r * n + col + c);
                v[k] = STREAM ? __builtin_nontemporal_load(p) : *p;
            }
        }
    };
    auto stage = [&](const f64x2 *v) {
#pragma unroll
        for (int k = 0; k < kBSteps; ++k) {
            t[r0 + k * kBRows][c] = v[k][0];
            t[r0 + k * kBRows][c + 1] = v[k][1];
        }
    };
    auto store = [&](int64_t row, int64_t col, const f64x2 *v) {  // v + the staged tile^T
#pragma unroll
        for (int k = 0; k < kBSteps; ++k) {
            const int64_t r = row + r0 + k * kBRows;
            if (r < n && col + c < n) {
                f64x2 o;
                o[0] = v[k][0] + t[c][r0 + k * kBRows];
                o[1] = v[k][1] + t[c + 1][r0 + k * kBRows];
                __builtin_nontemporal_store(o, (f64x2 *)(y + r * n + col + c));
            }
        }
    };
    f64x2 a[kBSteps], b[kBSteps];
    load(i0, j0, a);
    if (I == J) {
        stage(a);
        __syncthreads();
        store(i0, j0, a);
        return;
    }
    load(j0, i0, b);
    stage(b);
    __syncthreads();
    store(i0, j0, a);
    __syncthreads();
    stage(a);
    __syncthreads();
    store(j0, i0, b);
}

}  // namespace

hipError_t launch_transpose_sum(const double *x, double *y, int64_t n, hipStream_t s)
{
    if (n == 0)
        return hipSuccess;
    const int64_t B = (n + kBT - 1) / kBT, big = B * (B + 1) / 2;
    if (big >= kBigPairs && n % 2 == 0 && ((uintptr_t)x | (uintptr_t)y) % 16 == 0) {
        const auto fn =
            8 * n * n > kStreamBytes ? transpose_sum_big<true> : transpose_sum_big<false>;
        trace_begin("transpose_sum", s);
        hipLaunchKernelGGL(fn, dim3((unsigned)big), dim3(kBThreads), 0, s, x, y, n, B);
        trace_end("transpose_sum", s);
        return hipGetLastError();
    }
    const int64_t T = (n + kTT - 1) / kTT;
    const int64_t pairs = T * (T + 1) / 2;
    trace_begin("transpose_sum", s);
    hipLaunchKernelGGL(transpose_sum_tiles, dim3((unsigned)pairs), dim3(kTThreads), 0, s, x, y, n, T);
    trace_end("transpose_sum", s);
    return hipGetLastError();
}

}  // namespace mdx
