// Products with a sparse transition matrix F (eqn3; the six-neighbour model of eqn2 has
// seven entries per row), stored in CSR (row_ptr, col_idx, val). Every product is bound by
// the dense operand's HBM traffic, so each is one coalesced sweep over dense rows:
//   spmm_rows:       Y = alpha F A + beta1 C1 + beta2 C2       (row i of Y from the rows of A
//                                                               that F's row i names)
//   dense_sparse_t:  G = P F^T                                  (row k of P staged in LDS, each
//                                                               output G[k][j] gathers from it
//                                                               with F's row j)
//   spmv_rows:       y_b = F x_b for the rows x_b of a block
// With G = P F^T and then F G, F P F^T is formed without transposing anything.
#include "kf_internal.h"

#include <algorithm>

namespace kfmeg {

namespace {

constexpr int TPB = 256;

// A row's entries are read EB at a time, all loads of a batch in flight before the first product (an index past the
// row's end reads the last entry, whose product is left out), and added in order. One entry at a time each waits
// for the one before: at N = 1500 (18 MB in, 18 MB out) spmm_rows took 26 us, with batches 22, with stripes
// and two columns a lane 18; dense_sparse_t 34, with batches and two rows a workgroup 21.
constexpr int EB = 8;

// V columns a lane (every row is 16-byte aligned; it holds a column past an
// odd n, which is read and not stored). A wave takes a row of a stripe of columns, and workgroup b stripe b mod 8:
// workgroups go round the 8 XCDs, so an XCD reads its stripe of A alone, which stays in its L2 (2.3 MB at
// N = 1500), instead of almost every row of A.
constexpr int V = 2;
template <typename TY>
__global__ void spmm_rows_kernel(int n, int ncols, const int* rp, const int* ci, const double* v, const double* A,
                                 int64_t lda, double alpha, const double* C1, int64_t ldc1, double beta1,
                                 const double* C2, int64_t ldc2, double beta2, TY* Y, int64_t ldy) {
    typedef double vec __attribute__((ext_vector_type(V)));
    auto at = [](const double* p) { return *reinterpret_cast<const vec*>(p); };
    const int width = ((ncols + 7) / 8 + 15) / 16 * 16, j0 = (blockIdx.x & 7) * width, j1 = min(ncols, j0 + width);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    for (int i = (blockIdx.x >> 3) * (TPB / 64) + wave; i < n; i += (gridDim.x >> 3) * (TPB / 64)) {
        const int e0 = rp[i], e1 = rp[i + 1];
        for (int j = j0 + lane * V; j < j1; j += 64 * V) {
            double s[V] = {};
            for (int e = e0; e < e1; e += EB) {
                double w[EB];
                vec a[EB];
#pragma unroll
                for (int u = 0; u < EB; ++u) {
                    const int f = min(e + u, e1 - 1);
                    w[u] = v[f];
                    a[u] = at(A + (int64_t)ci[f] * lda + j);
                }
#pragma unroll
                for (int u = 0; u < EB; ++u)
                    if (e + u < e1) {
#pragma unroll
                        for (int c = 0; c < V; ++c) s[c] += w[u] * a[u][c];
                    }
            }
            vec c1 = 0.0, c2 = 0.0;
            if (C1) c1 = at(C1 + (int64_t)i * ldc1 + j);
            if (C2) c2 = at(C2 + (int64_t)i * ldc2 + j);
#pragma unroll
            for (int c = 0; c < V; ++c) {
                double y = alpha * s[c];
                if (C1) y += beta1 * c1[c];
                if (C2) y += beta2 * c2[c];
                if (j + c < j1) Y[(int64_t)i * ldy + j + c] = (TY)y;
            }
        }
    }
}

// One workgroup per R rows of P (grid-stride over rows), which share the reads of F; with STAGE the rows sit in
// dynamic LDS, otherwise (R = 1) the row is gathered from global memory (rows longer than the LDS budget).
template <int R, bool STAGE>
__global__ void dense_sparse_t_kernel(int n, const double* P, int64_t ldp, const int* rp, const int* ci,
                                      const double* v, double* G, int64_t ldg) {
    extern __shared__ double prow[];
    for (int k = blockIdx.x * R; k < n; k += gridDim.x * R) {
        const double* src = P + (int64_t)k * ldp;
        if constexpr (STAGE) {
            __syncthreads();
#pragma unroll
            for (int r = 0; r < R; ++r)
                for (int l = threadIdx.x; l < n; l += TPB) prow[r * n + l] = src[(int64_t)min(r, n - 1 - k) * ldp + l];
            __syncthreads();
        }
        for (int j = threadIdx.x; j < n; j += TPB) {
            double s[R] = {};
            const int e1 = rp[j + 1];
            for (int e = rp[j]; e < e1; e += EB) {
                double w[EB];
                int c[EB];
#pragma unroll
                for (int u = 0; u < EB; ++u) {
                    const int f = min(e + u, e1 - 1);
                    w[u] = v[f];
                    c[u] = ci[f];
                }
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    double a[EB];
#pragma unroll
                    for (int u = 0; u < EB; ++u) a[u] = STAGE ? prow[r * n + c[u]] : src[c[u]];
#pragma unroll
                    for (int u = 0; u < EB; ++u)
                        if (e + u < e1) s[r] += w[u] * a[u];
                }
            }
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (k + r < n) G[(int64_t)(k + r) * ldg + j] = s[r];
        }
    }
}

__global__ void spmv_rows_kernel(int n, int rows, const int* rp, const int* ci, const double* v, const double* X,
                                 int64_t ldx, double* Y, int64_t ldy) {
    for (int b = blockIdx.y; b < rows; b += gridDim.y)
        for (int i = blockIdx.x * TPB + threadIdx.x; i < n; i += gridDim.x * TPB) {
            double s = 0.0;
            for (int e = rp[i]; e < rp[i + 1]; ++e) s += v[e] * X[(int64_t)b * ldx + ci[e]];
            Y[(int64_t)b * ldy + i] = s;
        }
}

}  // namespace

hipError_t spmm_rows(const Csr& F, const double* A, int64_t lda, double alpha, const double* C1, int64_t ldc1,
                     double beta1, const double* C2, int64_t ldc2, double beta2, void* Y, bool y32, int64_t ldy,
                     hipStream_t s) {
    const int n = F.n;
    auto even = [](const void* p, int64_t ld) { return ((uintptr_t)p & 15) == 0 && ld % 2 == 0; };
    if (!even(A, lda) || !even(C1, C1 ? ldc1 : 0) || !even(C2, C2 ? ldc2 : 0)) return hipErrorInvalidValue;
    const dim3 grid((unsigned)(8 * std::max(1, std::min((n + TPB / 64 - 1) / (TPB / 64), 65535))));
    if (y32)
        hipLaunchKernelGGL(spmm_rows_kernel<float>, grid, dim3(TPB), 0, s, n, n, F.rp, F.ci, F.v, A, lda, alpha, C1,
                           ldc1, beta1, C2, ldc2, beta2, static_cast<float*>(Y), ldy);
    else
        hipLaunchKernelGGL(spmm_rows_kernel<double>, grid, dim3(TPB), 0, s, n, n, F.rp, F.ci, F.v, A, lda, alpha, C1,
                           ldc1, beta1, C2, ldc2, beta2, static_cast<double*>(Y), ldy);
    return hipGetLastError();
}

hipError_t dense_sparse_t(const Csr& F, const double* P, int64_t ldp, double* G, int64_t ldg, hipStream_t s) {
    const int n = F.n;
    const size_t lds = (size_t)n * sizeof(double);
    // two rows a workgroup while four workgroups still fit a compute unit
    if (2 * lds <= 32768)
        hipLaunchKernelGGL((dense_sparse_t_kernel<2, true>), dim3((unsigned)std::min((n + 1) / 2, 65535)), dim3(TPB),
                           2 * lds, s, n, P, ldp, F.rp, F.ci, F.v, G, ldg);
    else if (lds <= kMaxTransitionLds)
        hipLaunchKernelGGL((dense_sparse_t_kernel<1, true>), dim3((unsigned)std::min(n, 65535)), dim3(TPB), lds, s, n,
                           P, ldp, F.rp, F.ci, F.v, G, ldg);
    else
        hipLaunchKernelGGL((dense_sparse_t_kernel<1, false>), dim3((unsigned)std::min(n, 65535)), dim3(TPB), 0, s, n, P,
                           ldp, F.rp, F.ci, F.v, G, ldg);
    return hipGetLastError();
}

hipError_t spmv_rows(const Csr& F, const double* X, int64_t ldx, int rows, double* Y, int64_t ldy, hipStream_t s) {
    const int n = F.n;
    const dim3 grid((unsigned)std::max(1, (n + TPB - 1) / TPB), (unsigned)std::max(1, std::min(rows, 65535)));
    hipLaunchKernelGGL(spmv_rows_kernel, grid, dim3(TPB), 0, s, n, rows, F.rp, F.ci, F.v, X, ldx, Y, ldy);
    return hipGetLastError();
}

}  // namespace kfmeg
