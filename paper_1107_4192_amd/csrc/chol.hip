// Blocked Cholesky factorisation fused with the inverse of the factor (float64),
// for a batch of independent matrices.
//
// The filter needs S^{-1} in eqn8/eqn9, applied through the lower Cholesky
// factor L and its inverse Li = L^{-1}: S^{-1} B = Li^T (Li B). Li is obtained
// by solving L Z = I in the same right-looking sweep as the factorisation. The
// smoother's P_{t+1|t}^{-1} in eqn11 uses the same sweep only for the diagonal
// blocks of an outer-blocked factorisation (second half of this file).
//
// Two-level blocking keeps the O(n^3) work in large MFMA products with a long K dimension:
//   for each panel K (of kCholPanel columns):
//     for each 64-column block k of the panel, one launch of chol_step_kernel:
//       L_{>k,k} = A_{>k,k} Li_kk^T  and  Z_{k,<k} = Li_kk Z_{k,<k}, then inside the panel only
//       A_{>k,(k,K]} -= L_{>k,k} L_{(k,K],k}^T and Z_{(k,K],<=k} -= L_{(k,K],k} Z_{k,<=k}, and the
//       next diagonal block is factored and inverted, flagging a non-positive or non-finite pivot
//     trailing, K = the panel, one grouped GEMM launch:  A_{>K,>K} -= L_{>K,K} L_{>K,K}^T  and
//       Z_{>K,<=K} -= L_{>K,K} Z_{K,<=K}
// Every launch covers the whole batch, so the latency of the sequential sweep is shared by every
// matrix of the batch.
#include "kf_internal.h"

#include <algorithm>
#include <type_traits>

namespace kfmeg {

namespace {

constexpr int NB = 64;      // diagonal block
constexpr int NTD = 512;     // eight waves

struct DiagBatch {
    double* W[kMaxBatch];
    double* Z[kMaxBatch];
    int step[kMaxBatch];
};

typedef double d4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ d4 mfma(double a, double b, d4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// 64 x 64 tiles in LDS as rows of LD doubles: 66 puts the 32 lanes of a half wave that read one
// MFMA fragment (16 rows x 2 columns) on distinct bank pairs.
constexpr int LD = NB + 2;
constexpr int TILE = NB * LD;

// The value of lane L of each row of 16 lanes, in every lane of the row.
template <int L>
__device__ __forceinline__ double row_lane(double v) {
    const long long b = __double_as_longlong(v);
    return __longlong_as_double(__builtin_amdgcn_update_dpp(0LL, b, 0x150 + L, 0xf, 0xf, true));      // row_newbcast:L
}

// Tile of at most 64 x 64 (rows x cols valid, the rest zero, or the identity's with `unit`): into
// registers, and from there into LDS.
constexpr int TV = NB * NB / NTD;
__device__ __forceinline__ void fetch_tile(double (&v)[TV], const double* G, int64_t ldg, int rows, int cols, bool unit) {
    const int c = threadIdx.x & (NB - 1), g = threadIdx.x >> 6;
#pragma unroll
    for (int r = 0; r < TV; ++r) {
        const int i = g + NTD / 64 * r;
        v[r] = (i < rows && c < cols) ? G[(int64_t)i * ldg + c] : (unit && i == c ? 1.0 : 0.0);
    }
}
__device__ __forceinline__ void put_tile(double* S, const double (&v)[TV]) {
    const int c = threadIdx.x & (NB - 1), g = threadIdx.x >> 6;
#pragma unroll
    for (int r = 0; r < TV; ++r) S[(g + NTD / 64 * r) * LD + c] = v[r];
}

// acc (this wave's 32 x 16 part of a 64 x 64 tile as two MFMA blocks) = X Y, K = 64, with
// Y(k, j) = Y[k * sk + j * sj].
__device__ __forceinline__ void tile_mma(d4 (&acc)[2], const double* X, const double* Y, int sk, int sj) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int lr = lane & 15, lk = lane >> 4;
    const double* x0 = X + ((wave >> 2) * 32 + lr) * LD + lk;
    const double* y0 = Y + ((wave & 3) * 16 + lr) * sj + lk * sk;
    acc[0] = acc[1] = d4{0, 0, 0, 0};
#pragma unroll 4
    for (int k = 0; k < NB; k += 4) {
        const double a0 = x0[k], a1 = x0[16 * LD + k], b = y0[k * sk];
        acc[0] = mfma(a0, b, acc[0]);
        acc[1] = mfma(a1, b, acc[1]);
    }
}

// Row and column in the tile of element r of block x.
__device__ __forceinline__ int acc_row(int x, int r) {
    return (threadIdx.x >> 8) * 32 + 16 * x + ((threadIdx.x >> 4) & 3) + 4 * r;
}
__device__ __forceinline__ int acc_col() { return ((threadIdx.x >> 6) & 3) * 16 + (threadIdx.x & 15); }

// Cholesky factorisation and inverse of the 64 x 64 tile in S (512 threads; the lower triangle is
// read). Right-looking by columns: with d_j the pivot and c_ij = A_ij as column j comes up,
//     A_ik -= c_ij (c_kj / d_j)  (k > j)      U_ic -= c_ij (U_jc / d_j)  (c <= j < i, U = I at first)
// so L_ij = c_ij / sqrt(d_j) and (L^{-1})_ic = U_ic / sqrt(d_i). On return S holds c (columns j <= i), Z holds U and
// ys the 1 / sqrt(d): tile_l and tile_z scale them on the way out. Returns the first bad pivot's row, or NB.
//
// Bound by the chain of 64 pivots and, on the one wave that runs it, by the issue of a float64 instruction
// every 8 cycles. Blocks of 16 columns, one wave a block: a lane holds a row of the diagonal block (the same in each of
// its four rows of 16 lanes) and sixteen values of one of the other three blocks that the columns touch or of
// the identity: a row of the panel below or a column of U's rows. The multipliers reach the lanes by a DPP operand
// (row_newbcast), so a block needs no LDS, barrier or scalar register between its columns. What the next block reads is
// then updated by MFMA, one 16 x 16 tile each on four waves; the other tiles follow on the other waves
// beside the next block's columns. An MFMA adds its products one after the other in the order of k, each
// rounded, so the blocked form gives the bits of the plain column loop. 1/sqrt of a pivot is the hardware
// estimate refined by two Newton steps (accurate to a few ulp).
// Cycles for a tile: 24.5k (a block 4.9k, its MFMA step 1.2k). With panels of 8 columns, a row per lane, multipliers
// by readlane and all of the MFMA work between the panels: 44.4k. A launch that only factors: 14 us (23 before; 38
// with a barrier and LDS exchange per column).
constexpr int PB = 16;

// Columns K and, with N = 2, K + 1 take a column of the block's row (factor fa) and of the lane's other values
// (fx): m and c as the pivots' step below leaves them. The broadcast is part of the sum, which the compiler does not
// do by itself; the wait is that of a DPP operand after a vector instruction wrote it. What this writes is not read
// by a DPP operand before other instructions have rewritten it.
template <int K, int N>
__device__ __forceinline__ void fmac_bcast(double (&a)[PB], double (&x)[PB], double m, double c, double fa, double fx) {
    if constexpr (N == 1)
        asm volatile("s_nop 1\n\t"
                     "v_fmac_f64_dpp %0, %2, %4 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t"
                     "v_fmac_f64_dpp %1, %3, %5 row_newbcast:%6 row_mask:0xf bank_mask:0xf"
                     : "+&v"(a[K]), "+&v"(x[K])
                     : "v"(m), "v"(c), "v"(fa), "v"(fx), "n"(K));
    else
        asm volatile("s_nop 1\n\t"
                     "v_fmac_f64_dpp %0, %4, %6 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n\t"
                     "v_fmac_f64_dpp %1, %5, %7 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n\t"
                     "v_fmac_f64_dpp %2, %4, %6 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
                     "v_fmac_f64_dpp %3, %5, %7 row_newbcast:%9 row_mask:0xf bank_mask:0xf"
                     : "+&v"(a[K]), "+&v"(x[K]), "+&v"(a[K + 1]), "+&v"(x[K + 1])
                     : "v"(m), "v"(c), "v"(fa), "v"(fx), "n"(K), "n"(K + 1));
}
template <int K, int KE>
__device__ __forceinline__ void eliminate(double (&a)[PB], double (&x)[PB], double m, double c, double fa, double fx) {
    if constexpr (K < KE) {
        constexpr int N = K + 1 < KE ? 2 : 1;
        fmac_bcast<K, N>(a, x, m, c, fa, fx);
        eliminate<K + N, KE>(a, x, m, c, fa, fx);
    }
}
template <int J>
__device__ __forceinline__ void eliminate_from(double (&a)[PB], double (&x)[PB], double m0, double c0, double h0,
                                               bool isu, int lr, double& yl) {
    if constexpr (J < PB) {
        // the chain of pivot J, between its links the rest of column J - 1
        constexpr int R = PB - J - 1, Q = J > 0 ? J - 1 : 0;
        auto rest = [&](auto part) {
            constexpr int I = decltype(part)::value;
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (J > 0) eliminate<J + 1 + R * I / 3, J + 1 + R * (I + 1) / 3>(a, x, m0, c0, a[Q], h0);
            __builtin_amdgcn_sched_barrier(0);
        };
        const double d = row_lane<J>(a[J]);
        double y = __builtin_amdgcn_rsq(d);
        const double hd = 0.5 * d;
        rest(std::integral_constant<int, 0>());
        y = y * fma(-(hd * y), y, 1.5);
        rest(std::integral_constant<int, 1>());
        y = y * fma(-(hd * y), y, 1.5);
        rest(std::integral_constant<int, 2>());
        if (lr == J) yl = y;
        const double y2 = y * y, m = a[J] * -y2;
        // a row of the panel takes -c_ij (c_kj / d_j), a column of U takes c_kj (-U_jc / d_j)
        const double c = isu ? a[J] : m, h = isu ? x[J] * -y2 : x[J];
        if constexpr (J + 1 < PB) {                  // the next pivot's column first
            a[J + 1] = fma(row_lane<J + 1>(m), a[J], a[J + 1]);
            x[J + 1] = fma(row_lane<J + 1>(c), h, x[J + 1]);
        }
        eliminate_from<J + 1>(a, x, m, c, h, isu, lr, yl);
    }
}

__device__ __forceinline__ int potrf_inv_tile(double* S, double* Z, double* ys, double* inv2) {
    __shared__ int badrow;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, lk = lane >> 4;
    int bad = NB;
    // Block b applied to a 16 x 16 tile of S, or of the rows of U below the block.
    auto apply = [&](int b, bool inv, int ti, int tj) {
        const int c0 = PB * b, i = 16 * ti + lr, j = 16 * tj + lr;
        double* T = (inv ? Z : S) + (16 * ti + lk) * LD + j;
        const double* sx = S + i * LD + c0 + lk;
        const double* sy = inv ? Z + (c0 + lk) * LD + j : S + j * LD + c0 + lk;
        const int st = inv ? LD : 1;
        d4 acc;
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[r] = inv && tj == b ? 0.0 : T[4 * r * LD];
#pragma unroll
        for (int k = 0; k < PB; k += 4) acc = mfma(-sx[k], sy[k * st] * inv2[c0 + k + lk], acc);
#pragma unroll
        for (int r = 0; r < 4; ++r) T[4 * r * LD] = acc[r];
    };
#pragma unroll 1
    for (int b = 0; b < NB / PB; ++b) {
        const int c0 = PB * b;
        if (wave == 0) {
            // lanes of row lk: the block's row lr, and by lk against b a row of the panel, a column of U's
            // diagonal block (of I as yet) or a column of U's rows in an earlier block
            const bool isu = lk <= b;
            double* xp = isu ? Z + c0 * LD + 16 * lk + lr : S + (16 * lk + lr) * LD + c0;
            const int xs = isu ? LD : 1;
            double a[PB], x[PB];
#pragma unroll
            for (int k = 0; k < PB; ++k) {
                a[k] = S[(c0 + lr) * LD + c0 + k];
                x[k] = lk == b ? (lr == k ? 1.0 : 0.0) : xp[k * xs];
            }
            double yl = 0.0;
            eliminate_from<0>(a, x, 0.0, 0.0, 0.0, isu, lr, yl);
            // rows above a column hold no part of the lower triangle: whatever is there stays in its lane
#pragma unroll
            for (int k = 0; k < PB; ++k) {
                xp[k * xs] = x[k];
                if (lk == b) S[(c0 + lr) * LD + c0 + k] = a[k];
            }
            if (lk == b) {
                ys[c0 + lr] = yl;
                inv2[c0 + lr] = yl * yl;
            }
            // (1/sqrt comes out infinite or NaN exactly if the pivot is not positive or not finite)
            const unsigned long long off = __ballot(!isfinite(yl)) & 0xffff;
            if (off && bad == NB) bad = c0 + __ffsll(off) - 1;
        } else if (b > 0) {
            // beside it what block b - 1 does to the columns and rows after block b
            const int n1 = NB / PB - 1 - b, na = n1 * (n1 + 1) / 2;
#pragma unroll 1
            for (int u = wave - 1; u < na + n1 * b; u += NTD / 64 - 1) {
                int i = 0, j = u;
                if (u < na) while (j > i) { j -= i + 1; ++i; }
                else for (j -= na; j >= b; j -= b) ++i;
                apply(b - 1, u >= na, b + 1 + i, u < na ? b + 1 + j : j);
            }
        }
        __syncthreads();
        // block b applied to the next block's columns and rows: always four tiles
        if (b + 1 < NB / PB && wave < 4) {
            const bool inv = wave <= b;
            apply(b, inv, inv ? b + 1 : wave, inv ? wave : b + 1);
        }
        __syncthreads();
    }
    if (tid == 0) badrow = bad;
    __syncthreads();
    return badrow;
}

// L and L^{-1} from the tiles that potrf_inv_tile left, explicit zeros above the diagonal.
__device__ __forceinline__ double tile_l(const double* S, const double* ys, int i, int c) {
    return c <= i ? S[i * LD + c] * ys[c] : 0.0;
}
__device__ __forceinline__ double tile_z(const double* Z, const double* ys, int i, int c) {
    return c <= i ? Z[i * LD + c] * ys[i] : 0.0;
}

// One step of the sweep through the 64-column blocks [p0, p1) of a panel (blockIdx.y: matrix), block
// indices counted from the matrix's first. With column block c = k - 1 >= p0 factored (c_cc's L in W, Li_cc
// in Z), a workgroup takes one of
//   * a tile (i, j) of the panel's later columns, k <= j < p1, j <= i:  A_ij -= L_ic L_jc^T; the tile (k, k),
//     which comes first, is then factored and inverted on the spot;
//   * a tile (i, j) of the inverse, k <= i < p1, j <= c:  Z_ij -= L_ic Z_cj  (Z_ic = -L_ic Li_cc);
//   * tiles that no other workgroup of this launch reads, left by the launch before: column f = k - 2
//     of L in place, and Z_fj = Li_ff Z_fj, j < f,
// forming L_ic = A_ic Li_cc^T and Li_cc Z_cj itself: up to 3 products of 64^3 a tile where a separate
// panel pass would need 1, but no launch and no memory pass between the panel and the update. The
// sweep is bound by its chain (per launch two 64^3 products, 1.7 us each on one compute unit, and the
// factorisation of the next block), so the extra products cost nothing while the tiles fit the device.
// Launch k = p0 only factors (and at p0 = 0 clears Z off its diagonal blocks); launch k = p1 finishes columns
// and rows p1 - 2 and p1 - 1. A launch takes 19-21 us, one that only factors 14, one that only finishes 6 (one matrix of
// order 306 to 2000, nothing beside it). One launch per block instead of a factorisation, a panel and an
// update GEMM (8 launches at n = 306 where there were 16) took the filter's step at N = 5124, m = 306 from 1.04
// to 0.93 ms and a serving stream of six jobs of N = 2000 from 165 to 124 ms, at 33 us a launch.
__global__ __launch_bounds__(NTD) void chol_step_kernel(DiagBatch B, int64_t ldw, int64_t ldz, int n, int p0, int p1,
                                                        int k, DevStatus* status, int which, int row0) {
    __shared__ double S0[TILE], S1[TILE], ys[NB], inv2[NB];
    const int nblk = (n + NB - 1) / NB, c = k - 1;
    double* W = B.W[blockIdx.y];
    double* Z = B.Z[blockIdx.y];
    auto w = [&](int i, int j) { return W + (int64_t)i * NB * ldw + j * NB; };
    auto z = [&](int i, int j) { return Z + (int64_t)i * NB * ldz + j * NB; };
    auto ext = [&](int i) { return min(NB, n - i * NB); };
    const int cc = threadIdx.x & (NB - 1), g = threadIdx.x >> 6;
    int u = blockIdx.x;
    if (k == p0 && u > 0) {                          // p0 = 0: zeros off the diagonal blocks of Z
        --u;
        int i = u / (nblk - 1), j = u % (nblk - 1);
        if (j >= i) ++j;
        for (int r = g; r < ext(i); r += NTD / 64)
            if (cc < ext(j)) z(i, j)[(int64_t)r * ldz + cc] = 0.0;
        return;
    }
    // The tile's operands: a and l go to LDS, b waits in registers, so that two tiles of LDS are enough and a
    // workgroup fits beside one of the 128 x 128 products (64 KB) on a compute unit. L_ic = a l^T; b becomes
    // b l^T (a panel block) or l b (a block row of Z); the last product is X Y, subtracted from (add) or
    // stored to `out`.
    const double *ga = nullptr, *gb = nullptr, *gl = nullptr;
    int ra = NB, rb = NB, cb = NB, rl = NB, ro = NB, co = NB;
    int64_t lda = ldw, ldb = ldw, ldo = ldw;
    double* out = nullptr;
    const double *X = S0, *Y = S0;
    int sk = 1, sj = LD;                             // Y read as rows, Y(k, j) = Y[j][k]
    bool pa = false, pb = false, add = true, lb = false;
    const bool diag = u == 0 && k < p1;              // the next diagonal block
    const int q = p1 - k;                            // columns of the panel not yet factored
    const int nw = q * (nblk - k) - q * (q - 1) / 2, nz = k > p0 ? q * k : 0;
    if (u < nw || diag) {                            // tile of the panel's later columns
        int j = k, r = u;
        while (r >= nblk - j) { r -= nblk - j; ++j; }
        const int i = j + r;
        if (k > p0) {
            ga = w(i, c); ra = ext(i); gl = z(c, c);
            pa = true;
        }
        if (diag) {
            gb = w(k, k); rb = cb = ext(k);
        } else {
            if (i != j) { gb = w(j, c); rb = ext(j); pb = true; Y = S1; }
            out = w(i, j); ro = ext(i); co = ext(j);
        }
    } else if (u < nw + nz) {                        // tile (i, j) of the inverse, j < k <= i < p1
        const int i = k + (u - nw) / k, j = (u - nw) % k;
        ga = w(i, c); ra = ext(i); gl = z(c, c);
        pa = true;
        if (j < c) { gb = z(c, j); ldb = ldz; pb = lb = true; }
        else add = false;
        Y = S1; sk = LD; sj = 1;
        out = z(i, j); ldo = ldz; ro = ext(i);
    } else {
        // finish column f of L below it, then row f of Z (nblk - 1 tiles together); the last launch takes
        // f = p1 - 1 after f = p1 - 2
        u -= nw + nz;
        int f = k - 2;
        if (f < p0 || u >= nblk - 1) {
            if (f >= p0) u -= nblk - 1;
            f = p1 - 1;
        }
        gl = z(f, f); rl = ext(f);
        add = false;
        if (u < nblk - 1 - f) {                      // L_if = A_if Li_ff^T
            const int i = f + 1 + u;
            ga = w(i, f); ra = ext(i);
            Y = S1;
            out = w(i, f); ro = ext(i);
        } else {                                     // Z_fj = Li_ff Z_fj
            const int j = u - (nblk - 1 - f);
            ga = z(f, j); lda = ldz; ra = ext(f);
            X = S1; sk = LD; sj = 1;
            out = z(f, j); ldo = ldz; ro = ext(f);
        }
    }
    double va[TV], vb[TV], vl[TV];
    if (gl) fetch_tile(vl, gl, ldz, rl, rl, false);
    if (ga) fetch_tile(va, ga, lda, ra, NB, false);
    if (gb) fetch_tile(vb, gb, ldb, rb, cb, diag);
    if (gl) put_tile(S1, vl);
    if (ga) put_tile(S0, va);
    if (!gl) put_tile(S1, vb);                       // the first block of a panel: only to be factored
    __syncthreads();
    d4 acc[2], lic[2];
    const bool plain = !pa && !add;                  // a finishing tile: one product
    auto put_acc = [&](double* t, const d4 (&v)[2]) {
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int r = 0; r < 4; ++r) t[acc_row(a, r) * LD + acc_col()] = v[a][r];
    };
    if (pa) {
        tile_mma(lic, S0, S1, 1, LD);
        __syncthreads();
        if (pb) {
            put_tile(S0, vb);
            __syncthreads();
            tile_mma(acc, lb ? S1 : S0, lb ? S0 : S1, lb ? LD : 1, lb ? 1 : LD);
            __syncthreads();
            put_acc(S1, acc);
        } else if (diag) {
            put_tile(S1, vb);
        }
        put_acc(S0, lic);
        __syncthreads();
    }
    if (pa || !diag) tile_mma(acc, X, Y, sk, sj);
    // finishing tiles are the product itself; the others subtract it (a first touch of Z from zero)
    const double sgn = plain ? 1.0 : -1.0;
    if (!diag) {
        double old[2][4] = {};
        const int j = acc_col();
        if (add) {
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int i = acc_row(a, r);
                    if (i < ro && j < co) old[a][r] = out[(int64_t)i * ldo + j];
                }
        }
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = acc_row(a, r);
                if (i < ro && j < co) out[(int64_t)i * ldo + j] = old[a][r] + sgn * acc[a][r];
            }
        return;
    }
    if (pa) {
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int r = 0; r < 4; ++r) S1[acc_row(a, r) * LD + acc_col()] -= acc[a][r];
    }
    __syncthreads();
    const int bad = potrf_inv_tile(S1, S0, ys, inv2);
#pragma unroll 4
    for (int i = g; i < ext(k); i += NTD / 64) {
        if (cc >= ext(k)) continue;
        w(k, k)[(int64_t)i * ldw + cc] = tile_l(S1, ys, i, cc);
        z(k, k)[(int64_t)i * ldz + cc] = tile_z(S0, ys, i, cc);
    }
    if (threadIdx.x == 0 && bad < ext(k) && status)
        atomicMin(&status->key, status_key(B.step[blockIdx.y], row0 + k * NB + bad, which));
}

// Workgroups of launch k of the panel [p0, p1) of nblk blocks (the kernel's numbering; f < p1 as its
// columns and rows together are nblk - 1 tiles).
int step_tiles(int nblk, int p0, int p1, int k) {
    if (k == p0) return 1 + (p0 == 0 ? nblk * (nblk - 1) : 0);
    const int q = p1 - k;
    int t = q * (nblk - k) - q * (q - 1) / 2 + q * k;
    if (k - 2 >= p0) t += nblk - 1;
    if (k == p1) t += nblk - 1;
    return t;
}

}  // namespace

hipError_t chol_inv_batch(int n, double* const* W, int64_t ldw, double* const* Z, int64_t ldz, int count,
                          DevStatus* status, int which, const int* steps, hipStream_t s, int row_base, int panel) {
    if (panel < NB || panel % NB || count < 1 || count > kMaxBatch || n < 1) return hipErrorInvalidValue;
    hipError_t e;
    auto w = [&](int b, int i, int j) { return W[b] + (int64_t)i * ldw + j; };
    auto z = [&](int b, int i, int j) { return Z[b] + (int64_t)i * ldz + j; };
    DiagBatch db;
    for (int b = 0; b < count; ++b) {
        db.W[b] = W[b];
        db.Z[b] = Z[b];
        db.step[b] = steps ? steps[b] : 0;
    }
    const int nblk = (n + NB - 1) / NB;
    for (int c0 = 0; c0 < n; c0 += panel) {
        const int r2 = c0 + (n - c0 < panel ? n - c0 : panel);
        const int p0 = c0 / NB, p1 = (r2 + NB - 1) / NB;
        for (int k = p0; k <= p1; ++k) {
            const int tiles = step_tiles(nblk, p0, p1, k);
            if (tiles == 0) continue;     // nothing to finish: a single block
            hipLaunchKernelGGL(chol_step_kernel, dim3(tiles, count), dim3(NTD), 0, s, db, ldw, ldz, n, p0, p1, k, status,
                               which, row_base);
            if ((e = hipGetLastError()) != hipSuccess) return e;
        }
        if (r2 < n) {                     // trailing update with K = the panel width
            GemmProblem pr[kMaxGroup];
            int np = 0;
            for (int b = 0; b < count; ++b) {
                GemmProblem t1, t2;
                t1.M = n - r2; t1.N = n - r2; t1.K = r2 - c0;
                t1.A = w(b, r2, c0); t1.lda = ldw;
                t1.B = w(b, r2, c0); t1.ldb = ldw;
                t1.flags = G_TB | G_LOWER;
                t1.alpha = -1.0; t1.beta = 1.0;
                t1.Cin = w(b, r2, r2); t1.ldcin = ldw;
                t1.C = w(b, r2, r2); t1.ldc = ldw;
                t2.M = n - r2; t2.N = r2; t2.K = r2 - c0;
                t2.A = w(b, r2, c0); t2.lda = ldw;
                t2.B = z(b, c0, 0); t2.ldb = ldz;
                t2.alpha = -1.0; t2.beta = 1.0;
                t2.Cin = z(b, r2, 0); t2.ldcin = ldz;
                t2.C = z(b, r2, 0); t2.ldc = ldz;
                pr[np++] = t1;
                pr[np++] = t2;
            }
            if ((e = gemm_launch(Dt::F64, pr, np, s)) != hipSuccess) return e;
        }
    }
    return hipSuccess;
}

hipError_t chol_inv(double* W, int64_t ldw, double* Z, int64_t ldz, int n, DevStatus* status, int which,
                    int step, hipStream_t s, bool one_panel) {
    const int panel = one_panel && n <= kOnePanel ? kOnePanel : kCholPanel;
    return chol_inv_batch(n, &W, ldw, &Z, ldz, 1, status, which, &step, s, 0, panel);
}

// ------------------------------------------------------------------ outer-blocked factorisation and solves
// For the smoother gain (eqn11) the inverse of the whole factor is not needed: with L from an
// outer-blocked Cholesky of P_{t+1|t} (diagonal blocks of width nb factored and inverted by
// chol_inv_batch above), A_t^T = L^{-T} (L^{-1} F P_{t|t}) is two blocked triangular solves whose
// off-diagonal work is products with K up to n, and whose diagonal blocks are applied as products
// with the small inverses Li_kk. Every launch covers the whole batch.

namespace {

// The gain's products run as their own named kernel instantiation (profiling).
hipError_t gain_launch(GemmProblem* pr, int count, hipStream_t s) {
    for (int u = 0; u < count; ++u) pr[u].flags |= G_GAIN;
    return gemm_launch(Dt::F64, pr, count, s);
}

// Outer blocks of width nb; a remainder narrower than nb / 4 joins the last full block (so the
// last block is up to gain_block_width(n, nb) wide) rather than costing a sweep of its own.
struct Blocks {
    int n, nb;
    int count() const {
        const int full = n / nb, rem = n - full * nb;
        if (full == 0) return 1;
        return (rem == 0 || rem < nb / 4) ? full : full + 1;
    }
    int lo(int k) const { return k * nb; }
    int hi(int k) const { return k == count() - 1 ? n : (k + 1) * nb; }
};

}  // namespace

int gain_block_width(int n, int nb) {
    const Blocks bl{n, nb};
    return bl.hi(bl.count() - 1) - bl.lo(bl.count() - 1) > nb ? bl.hi(bl.count() - 1) - bl.lo(bl.count() - 1)
                                                               : std::min(n, nb);
}

hipError_t chol_blocked_batch(int n, int nb, double* const* W, int64_t ldw, double* const* D, int64_t ldd,
                              double* const* Tb, int64_t ldt, int count, DevStatus* status, int which,
                              const int* steps, hipStream_t s, const double* const* Pa, const double* Qa) {
    if (count < 1 || count > kMaxBatch || nb < 1 || ldd < gain_block_width(n, nb) || ldt < n || (!Pa != !Qa))
        return hipErrorInvalidValue;
    const Blocks bl{n, nb};
    hipError_t e;
    if (Pa) {   // the first block column of Pa + Qa (diagonal block and panel); the rest comes in below
        for (int b = 0; b < count; ++b)
            if ((e = axpby3(n, bl.hi(0), W[b], false, ldw, Pa[b], false, ldw, Qa, false, ldw, 1.0, nullptr, false,
                            0, 0.0, s)) != hipSuccess)
                return e;
    }
    for (int k = 0; k < bl.count(); ++k) {
        const int r0 = bl.lo(k), r1 = bl.hi(k), nbk = r1 - r0, nr = n - r1;
        double* Wd[kMaxBatch];
        double* Dd[kMaxBatch];
        for (int b = 0; b < count; ++b) {
            Wd[b] = W[b] + (int64_t)r0 * ldw + r0;
            Dd[b] = D[b] + (int64_t)r0 * ldd;
        }
        // L_kk and Li_kk of the diagonal block (its trailing part already updated)
        if ((e = chol_inv_batch(nbk, Wd, ldw, Dd, ldd, count, status, which, steps, s, r0)) != hipSuccess) return e;
        if (nr == 0) break;
        GemmProblem pr[kMaxGroup];
        for (int b = 0; b < count; ++b) {     // panel, transposed: Tb = Li_kk A_{>k,k}^T = L_{>k,k}^T
            GemmProblem& g = pr[b];
            g.M = nbk; g.N = nr; g.K = nbk;
            g.A = Dd[b]; g.lda = ldd; g.flags = G_ALOWER | G_TB;
            g.B = W[b] + (int64_t)r1 * ldw + r0; g.ldb = ldw;
            g.C = Tb[b]; g.ldc = ldt;
        }
        if ((e = gain_launch(pr, count, s)) != hipSuccess) return e;
        for (int b = 0; b < count; ++b) {     // trailing: A_{>k,>k} -= L_{>k,k} L_{>k,k}^T  (lower tiles)
            GemmProblem& g = pr[b];
            g = GemmProblem();
            g.M = nr; g.N = nr; g.K = nbk;
            g.A = Tb[b]; g.lda = ldt; g.flags = G_TA | G_LOWER;
            g.B = Tb[b]; g.ldb = ldt;
            g.alpha = -1.0; g.beta = 1.0;
            if (Pa && k == 0) {   // (Pa + Qa)_{>0,>0} - L L^T
                g.Cin = Pa[b] + (int64_t)r1 * ldw + r1; g.ldcin = ldw;
                g.Cin2 = Qa + (int64_t)r1 * ldw + r1; g.ldcin2 = ldw; g.gamma = 1.0;
            } else {
                g.Cin = W[b] + (int64_t)r1 * ldw + r1; g.ldcin = ldw;
            }
            g.C = W[b] + (int64_t)r1 * ldw + r1; g.ldc = ldw;
        }
        if ((e = gain_launch(pr, count, s)) != hipSuccess) return e;
        TransposeBatch tb;                    // the panel into place: W[r1 + i][r0 + c] = Tb[c][i]
        for (int b = 0; b < count; ++b) {
            tb.src[b] = Tb[b];
            tb.dst[b] = W[b] + (int64_t)r1 * ldw + r0;
            tb.dst32[b] = nullptr;
        }
        if ((e = transpose_batch(tb, count, nbk, nr, ldt, ldw, s)) != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t trsm_lower_batch(int n, int nb, const double* const* W, int64_t ldw, const double* const* D, int64_t ldd,
                            double* const* Tb, int64_t ldt, const double* const* B, int64_t ldb, double* const* Y,
                            int64_t ldy, int count, hipStream_t s) {
    if (count < 1 || count > kMaxBatch || ldt < n) return hipErrorInvalidValue;
    const Blocks bl{n, nb};
    hipError_t e;
    GemmProblem pr[kMaxGroup];
    for (int k = 0; k < bl.count(); ++k) {
        const int r0 = bl.lo(k), nbk = bl.hi(k) - r0;
        if (k > 0) {                          // Tb = B_k - L_{k,<k} Y_{<k}
            for (int b = 0; b < count; ++b) {
                GemmProblem& g = pr[b];
                g = GemmProblem();
                g.M = nbk; g.N = n; g.K = r0;
                g.A = W[b] + (int64_t)r0 * ldw; g.lda = ldw;
                g.B = Y[b]; g.ldb = ldy;
                g.alpha = -1.0; g.beta = 1.0;
                g.Cin = B[b] + (int64_t)r0 * ldb; g.ldcin = ldb;
                g.C = Tb[b]; g.ldc = ldt;
            }
            if ((e = gain_launch(pr, count, s)) != hipSuccess) return e;
        }
        for (int b = 0; b < count; ++b) {     // Y_k = Li_kk (B_k - ...)
            GemmProblem& g = pr[b];
            g = GemmProblem();
            g.M = nbk; g.N = n; g.K = nbk;
            g.A = D[b] + (int64_t)r0 * ldd; g.lda = ldd; g.flags = G_ALOWER;
            if (k > 0) { g.B = Tb[b]; g.ldb = ldt; }
            else { g.B = B[b]; g.ldb = ldb; }
            g.C = Y[b] + (int64_t)r0 * ldy; g.ldc = ldy;
        }
        if ((e = gain_launch(pr, count, s)) != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t trsm_upper_t_batch(int n, int nb, const double* const* W, int64_t ldw, const double* const* D,
                              int64_t ldd, double* const* Tb, int64_t ldt, const double* const* Y, int64_t ldy,
                              double* const* Z, int64_t ldz, int count, hipStream_t s) {
    if (count < 1 || count > kMaxBatch || ldt < n) return hipErrorInvalidValue;
    const Blocks bl{n, nb};
    hipError_t e;
    GemmProblem pr[kMaxGroup];
    for (int k = bl.count() - 1; k >= 0; --k) {
        const int r0 = bl.lo(k), r1 = bl.hi(k), nbk = r1 - r0;
        if (r1 < n) {                         // Tb = Y_k - L_{>k,k}^T Z_{>k}
            for (int b = 0; b < count; ++b) {
                GemmProblem& g = pr[b];
                g = GemmProblem();
                g.M = nbk; g.N = n; g.K = n - r1;
                g.A = W[b] + (int64_t)r1 * ldw + r0; g.lda = ldw; g.flags = G_TA;
                g.B = Z[b] + (int64_t)r1 * ldz; g.ldb = ldz;
                g.alpha = -1.0; g.beta = 1.0;
                g.Cin = Y[b] + (int64_t)r0 * ldy; g.ldcin = ldy;
                g.C = Tb[b]; g.ldc = ldt;
            }
            if ((e = gain_launch(pr, count, s)) != hipSuccess) return e;
        }
        for (int b = 0; b < count; ++b) {     // Z_k = Li_kk^T (Y_k - ...)
            GemmProblem& g = pr[b];
            g = GemmProblem();
            g.M = nbk; g.N = n; g.K = nbk;
            g.A = D[b] + (int64_t)r0 * ldd; g.lda = ldd; g.flags = G_TA | G_AUPPER;
            if (r1 < n) { g.B = Tb[b]; g.ldb = ldt; }
            else { g.B = Y[b] + (int64_t)r0 * ldy; g.ldb = ldy; }
            g.C = Z[b] + (int64_t)r0 * ldz; g.ldc = ldz;
        }
        if ((e = gain_launch(pr, count, s)) != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace kfmeg
