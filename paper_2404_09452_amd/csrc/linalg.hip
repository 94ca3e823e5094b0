// Dense FP64 linear algebra on the auxiliary metric, gfx950:
//   - blocked right-looking Cholesky V = L L^T (64-wide panels; the diagonal
//     block is factored and inverted by one workgroup; the panel below is
//     multiplied by that inverse and the trailing matrix updated, both on FP64
//     MFMA),
//   - L^{-1} by blocked forward substitution on the identity, block row by
//     block row (row i needs only the factor steps up to i),
//   - the whitening B = U L^{-T}-transposed product, i.e. B[f][P] =
//     sum_{Q<=P} U[f][Q] Linv[P][Q], as one MFMA GEMM that stops each output
//     tile's k loop at its last column (Linv is lower triangular).
// Matrices are row-major with the padded leading dimension npad (a multiple
// of 64); the pad block of the metric is the identity so every factor stays
// well defined and the pad rows/columns of B are exactly zero.
#include <climits>

#include "dfjk_internal.h"
#include "mfma_f64.h"

namespace dfjk {

constexpr int NBK = 64;   // panel width

__global__ void k_metric_pad(double *V, int64_t n, int64_t npad)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= npad * npad) return;
    const int64_t r = i / npad, c = i % npad;
    if (r >= n || c >= n) V[i] = (r == c) ? 1.0 : 0.0;
}

void launch_metric_pad(double *V, int64_t n, int64_t npad, hipStream_t s)
{
    const int64_t tot = npad * npad;
    hipLaunchKernelGGL(k_metric_pad, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, V, n, npad);
}

// Lane `src`'s value of v, broadcast to the wave (two 32-bit lane reads).
__device__ __forceinline__ double readlane_f64(double v, int src)
{
    const long long bits = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)bits, src);
    const int hi = __builtin_amdgcn_readlane((int)(bits >> 32), src);
    return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

// Factor the 64x64 diagonal block at (k0, k0) in place and invert the factor, one
// workgroup of four waves.  What bounds it is a chain of dependent FP64 operations,
// so the block is taken in four panels of 16 columns:
//   - one wave factors a panel, lane i holding row i of it.  The steps run on
//     A = L' P L'^T (u_l u_i / pivot: one division in the chain); the square roots of the
//     16 pivots are taken at once, one lane each, and scale the columns at the end;
//   - the columns right of the panel are updated by all waves on FP64 MFMA;
//   - afterwards each wave inverts one 16x16 diagonal block (a column a lane), and
//     the blocks below follow by distance s from the diagonal, on MFMA:
//     X_ij = -X_ii sum_{k=j}^{i-1} L_ik X_kj; an accumulator has the layout of
//     the B operand, so the sum goes straight into the second product.
// One wave with a row a lane and no panels took 46 us; this takes 21.
// A pivot <= 0 is recorded (smallest index wins) and replaced by 1 so the remaining
// steps stay finite; the host reports the recorded index.
constexpr int PB = 16, LDB = NBK + 1;

__global__ __launch_bounds__(256) void k_potrf_diag(double *A, int64_t ld, int64_t k0, int32_t *status, double *Dk)
{
    __shared__ double S[NBK * LDB];     // the block, then L
    __shared__ double X[NBK * LDB];     // L^{-1}
    __shared__ double rdiag[NBK];       // 1 / L_jj
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int fr = lane & 15, fk = lane >> 4;   // MFMA operand row (column) and k
    double *blk = A + k0 * ld + k0;
    double v[NBK * NBK / 256];   // all loads in flight before the first is stored
#pragma unroll
    for (int i = 0; i < NBK * NBK / 256; ++i) v[i] = blk[(int64_t)(wave + 4 * i) * ld + lane];
#pragma unroll
    for (int i = 0; i < NBK * NBK / 256; ++i) {
        S[(wave + 4 * i) * LDB + lane] = v[i];
        X[(wave + 4 * i) * LDB + lane] = 0.0;
    }
    __syncthreads();
#pragma unroll 1
    for (int c0 = 0; c0 < NBK; c0 += PB) {
        if (wave == 0) {
            double r[PB], piv = 1.0;
            int bad = INT_MAX;
#pragma unroll
            for (int c = 0; c < PB; ++c) r[c] = S[lane * LDB + c0 + c];
#pragma unroll
            for (int j = 0; j < PB; ++j) {
                double d = readlane_f64(r[j], c0 + j);
                const bool ok = d > 0.0;
                bad = ok ? bad : min(bad, (int)(k0 + c0 + j));
                d = ok ? d : 1.0;
                piv = lane == c0 + j ? d : piv;
                // u / d: the hardware's estimate of 1 / d, two Newton steps and one of the quotient
                // (half the chain of a division, and exactly 1 for u = d: a repeated function
                // leaves a pivot of 0, not a rounding error of either sign)
                double q = __builtin_amdgcn_rcp(d);
                q = fma(q, fma(-d, q, 1.0), q);
                q = fma(q, fma(-d, q, 1.0), q);
                double w = r[j] * q;
                w = -fma(fma(-d, w, r[j]), q, w);
#pragma unroll
                for (int l = j + 1; l < PB; ++l) r[l] = fma(w, readlane_f64(r[j], c0 + l), r[l]);
            }
            if (lane == 0 && bad != INT_MAX) atomicMin(status, bad);
            const double root = sqrt(piv), inv = 1.0 / root;
            if (lane >= c0 && lane < c0 + PB) rdiag[lane] = inv;
#pragma unroll
            for (int j = 0; j < PB; ++j) {
                const double l = r[j] * readlane_f64(inv, c0 + j);
                r[j] = lane > c0 + j ? l : lane == c0 + j ? root : 0.0;
            }
            if (lane >= c0)
#pragma unroll
                for (int j = 0; j < PB; ++j) S[lane * LDB + c0 + j] = r[j];
        }
        __syncthreads();
        // S(ti, tj) -= L(ti, panel) L(tj, panel)^T for the tiles right of the panel
        const int n = (NBK - c0) / PB - 1;
        for (int t = wave; t < n * (n + 1) / 2; t += 4) {
            const int ri = t < 1 ? 0 : t < 3 ? 1 : 2, rj = t - ri * (ri + 1) / 2;
            const int i0 = c0 + PB * (ri + 1), j0 = c0 + PB * (rj + 1);
            f64x4 acc;
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[q] = S[(i0 + 4 * q + fk) * LDB + j0 + fr];
#pragma unroll
            for (int ks = 0; ks < PB; ks += 4)
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-S[(i0 + fr) * LDB + c0 + ks + fk],
                                                           S[(j0 + fr) * LDB + c0 + ks + fk], acc, 0, 0, 0);
#pragma unroll
            for (int q = 0; q < 4; ++q) S[(i0 + 4 * q + fk) * LDB + j0 + fr] = acc[q];
        }
        __syncthreads();
    }
    // entries above the diagonal blocks were never written: zero in L
    for (int e = tid; e < NBK * NBK; e += 256) {
        const int r = e >> 6, c = e & 63;
        blk[(int64_t)r * ld + c] = c <= r ? S[r * LDB + c] : 0.0;
    }
    if (lane < PB) {
        const int b0 = wave * PB;
        double x[PB];
#pragma unroll
        for (int q = 0; q < PB; ++q) x[q] = q == lane ? 1.0 : 0.0;
#pragma unroll
        for (int l = 0; l < PB; ++l) {
            x[l] *= rdiag[b0 + l];
#pragma unroll
            for (int q = l + 1; q < PB; ++q) x[q] = fma(-S[(b0 + q) * LDB + b0 + l], x[l], x[q]);
        }
#pragma unroll
        for (int q = 0; q < PB; ++q) X[(b0 + q) * LDB + b0 + lane] = x[q];
    }
    __syncthreads();
#pragma unroll 1
    for (int dist = 1; dist < NBK / PB; ++dist) {
        const int i0 = (wave + dist) * PB, j0 = wave * PB;
        if (wave + dist < NBK / PB) {
            f64x4 sum = {0.0, 0.0, 0.0, 0.0}, x = {0.0, 0.0, 0.0, 0.0};
            for (int k = j0; k < i0; k += 4)
                sum = __builtin_amdgcn_mfma_f64_16x16x4f64(S[(i0 + fr) * LDB + k + fk], X[(k + fk) * LDB + j0 + fr],
                                                           sum, 0, 0, 0);
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
                x = __builtin_amdgcn_mfma_f64_16x16x4f64(-X[(i0 + fr) * LDB + i0 + 4 * ks + fk], sum[ks], x, 0, 0, 0);
#pragma unroll
            for (int q = 0; q < 4; ++q) X[(i0 + 4 * q + fk) * LDB + j0 + fr] = x[q];
        }
        __syncthreads();
    }
    for (int e = tid; e < NBK * NBK; e += 256) Dk[e] = X[(e >> 6) * LDB + (e & 63)];
}

// One 64x64 tile of C = A Bop or (SUB) C -= A Bop over k = 64, Bop(k, n) = B[n][k] or
// (NN) B[k][n]: the products of the factor and of the inverse.  Every size is a
// multiple of 64.  Each of these launches is a few microseconds of latency (its
// operands come from other XCDs' last launch, past L2), so a workgroup asks for both
// operands and its part of C at once and meets one barrier: 5 us, where the general
// tile kernel, staging k by 16 and reading C last, took 7 (C = A Bop) and 11 (SUB).
// In place where a tile reads only its own 64 rows or columns of C: they are all in
// LDS before the first write.
struct StepArgs {
    const double *A, *B;
    double *C;
    int64_t lda, ldb, ldc;
    int32_t ntm, lower;   // tiles down; lower: only tn <= tm
};

template <bool NN, bool SUB>
__global__ __launch_bounds__(256) void k_step(StepArgs g)
{
    constexpr int LDT = NBK + 2;   // 16-byte aligned rows, fragment reads in distinct banks
    __shared__ __align__(16) double As[NBK * LDT];
    __shared__ __align__(16) double Bs[NBK * LDT];
    int tm = (int)blockIdx.x % g.ntm, tn = (int)blockIdx.x / g.ntm;
    if (g.lower) {
        const int t = blockIdx.x;
        tm = (int)((sqrt(8.0 * t + 1.0) - 1.0) * 0.5);
        while (tm * (tm + 1) / 2 > t) --tm;
        while ((tm + 1) * (tm + 2) / 2 <= t) ++tm;
        tn = t - tm * (tm + 1) / 2;
    }
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int fr = lane & 15, fk = lane >> 4, wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
    const double *A = g.A + (int64_t)tm * NBK * g.lda;
    const double *B = NN ? g.B + (int64_t)tn * NBK : g.B + (int64_t)tn * NBK * g.ldb;
    double *C = g.C + ((int64_t)tm * NBK + wm + fk) * g.ldc + (int64_t)tn * NBK + wn + fr;
    double2 va[8], vb[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int r = (tid >> 5) + 8 * i, c = 2 * (tid & 31);
        va[i] = *reinterpret_cast<const double2 *>(A + r * g.lda + c);
        vb[i] = *reinterpret_cast<const double2 *>(B + r * g.ldb + c);
    }
    f64x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[i][j][q] = SUB ? C[(16 * i + 4 * q) * g.ldc + 16 * j] : 0.0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int r = (tid >> 5) + 8 * i, c = 2 * (tid & 31);
        if (SUB) va[i] = make_double2(-va[i].x, -va[i].y);
        *reinterpret_cast<double2 *>(As + r * LDT + c) = va[i];
        *reinterpret_cast<double2 *>(Bs + r * LDT + c) = vb[i];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NBK; k += 4) {
        double a[2], b[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            a[i] = As[(wm + 16 * i + fr) * LDT + k + fk];
            b[i] = NN ? Bs[(k + fk) * LDT + wn + 16 * i + fr] : Bs[(wn + 16 * i + fr) * LDT + k + fk];
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) C[(16 * i + 4 * q) * g.ldc + 16 * j] = acc[i][j][q];
}

// Step k of the blocked Cholesky: factor and invert the diagonal block,
// form the panel below it, update the trailing matrix.
void cholesky_step(double *A, int64_t npad, int64_t k, int32_t *status, double *Dinv, hipStream_t s)
{
    const int rest = (int)(npad / NBK - k - 1);
    const int64_t k0 = k * NBK, t0 = k0 + NBK;
    double *Dk = Dinv + k * NBK * NBK;
    hipLaunchKernelGGL(k_potrf_diag, dim3(1), dim3(256), 0, s, A, npad, k0, status, Dk);
    if (rest == 0) return;
    // panel: L21 = A21 L_kk^{-T} = A21 Dk^T, in place (each tile reads only its own rows)
    double *P = A + t0 * npad + k0;
    hipLaunchKernelGGL((k_step<false, false>), dim3(rest), dim3(256), 0, s,
                       StepArgs{P, Dk, P, npad, NBK, npad, rest, 0});
    // A22 -= L21 L21^T on the lower tiles of the trailing matrix
    hipLaunchKernelGGL((k_step<false, true>), dim3(rest * (rest + 1) / 2), dim3(256), 0, s,
                       StepArgs{P, P, A + t0 * npad + t0, npad, npad, npad, rest, 1});
}

void launch_cholesky(double *A, int64_t npad, int32_t *status, double *Dinv, hipStream_t s)
{
    for (int64_t k = 0; k < npad / NBK; ++k) cholesky_step(A, npad, k, status, Dinv, s);
}

__global__ void k_zero_upper(double *A, int64_t npad)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= npad * npad) return;
    if (i % npad > i / npad) A[i] = 0.0;
}

__global__ void k_identity(double *A, int64_t npad)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= npad * npad) return;
    A[i] = (i % npad == i / npad) ? 1.0 : 0.0;
}

void launch_zero_upper(double *L, int64_t npad, hipStream_t s)
{
    const int64_t tot = npad * npad;
    hipLaunchKernelGGL(k_zero_upper, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, L, npad);
}

void trtri_begin(double *X, int64_t npad, hipStream_t s)
{
    const int64_t tot = npad * npad;
    hipLaunchKernelGGL(k_identity, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, X, npad);
}

// X = L^{-1} by blocked forward substitution on the identity, block row i at
// a time: X_i[0:w] <- D_i X_i[0:w] (w = (i+1) 64, D_i = L_ii^{-1} from the
// factor's diagonal step; in place: each tile reads only its own block of X_i), then
// X[rows below][0:w] -= L[rows below][block i] X_i[0:w].  Step i reads only
// what Cholesky steps 0..i have finished (D_i and the strictly lower column
// block i of L), so it can follow step i on another stream.
void trtri_step(const double *L, double *X, const double *Dinv, int64_t npad, int64_t i, hipStream_t s)
{
    const int rest = (int)(npad / NBK - i - 1), cols = (int)i + 1;
    const int64_t i0 = i * NBK, w = i0 + NBK;
    double *Xi = X + i0 * npad;
    hipLaunchKernelGGL((k_step<true, false>), dim3(cols), dim3(256), 0, s,
                       StepArgs{Dinv + i * NBK * NBK, Xi, Xi, NBK, npad, npad, 1, 0});
    if (rest == 0) return;
    hipLaunchKernelGGL((k_step<true, true>), dim3(rest * cols), dim3(256), 0, s,
                       StepArgs{L + w * npad + i0, Xi, X + w * npad, npad, npad, npad, rest, 0});
}

// L^{-1} after the whole factor (Dinv as launch_cholesky left it); the upper
// triangle of L is zeroed for the callers that read L itself.
void launch_trtri(double *L, double *X, const double *Dinv, int64_t npad, hipStream_t s)
{
    launch_zero_upper(L, npad, s);
    trtri_begin(X, npad, s);
    for (int64_t i = 0; i < npad / NBK; ++i) trtri_step(L, X, Dinv, npad, i, s);
}

void launch_whiten(const double *U, const double *Linv, double *B, int64_t nf_pad, int64_t npad, hipStream_t s)
{
    launch_gemm_nt_tri(U, Linv, B, nf_pad, npad, npad, s);
}

}  // namespace dfjk
