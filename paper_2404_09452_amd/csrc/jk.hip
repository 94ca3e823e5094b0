// One DF-J/K build on gfx950, from the resident whitened tensor B[f][P]
// (f = stored AO function pair of a significant shell pair, P = aux function,
// row length naux_pad):
//   1. D = 2 C C^T                           (C route only)
//   2. c_P = sum_f d_f B[f][P], d_f = w_f D[mu_f][nu_f] (w = 2 for a != b blocks, 1
//      for a == a)                           split over f, fixed-order sum
//   3. J[mu_f][nu_f] = sum_P B[f][P] c_P     one wave per row f
//   4. X[mu][P][i] = sum_nu B[f(mu,nu)][P] C[nu][i]
//                                            gathered GEMM on FP64 MFMA, one
//                                            workgroup per (mu, 128 aux rows)
//   5. K = 2 X X^T (C route) or X B~^T (D route) on FP64 MFMA, lower tiles,
//      split-K into partial tiles summed in a fixed order
//   6. E_J = 1/2 sum_P c_P^2 (= 1/2 Tr DJ), E_K = -1/4 sum D K
// No floating-point atomics anywhere, so results are bitwise reproducible.
#include "dfjk_internal.h"
#include "mfma_f64.h"

#include <algorithm>

namespace dfjk {


constexpr int kCSplitRows = 512; // f rows per partial of c
constexpr double kAutoSlabBytes = 48e9;  // automatic aux slab: slab-sized K buffers up to this
constexpr double kPartBytes = 6e9;       // FP32 parts while the partial tiles of all slabs stay within this
constexpr double kJSideBytes = 64e6;     // J beside K from this size of B on (below, the fork costs more)

// ---------------------------------------------------------------------------
__global__ void k_fill(double *p, int64_t n, double v)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}
static void fill(double *p, int64_t n, double v, hipStream_t s)
{
    hipLaunchKernelGGL(k_fill, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n, v);
}

// D = scale C C^T, one thread per element of a 16x16 output block (block bx, by).
__device__ __forceinline__ void density_block(const double *__restrict__ C, int64_t nao, int32_t nocc, double scale,
                                              double *__restrict__ D, unsigned bx, unsigned by)
{
    __shared__ double Ca[16][65], Cb[16][65];
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    const int64_t m0 = (int64_t)by * 16, n0 = (int64_t)bx * 16;
    double s = 0.0;
    for (int i0 = 0; i0 < nocc; i0 += 64) {
        for (int e = threadIdx.x; e < 16 * 64; e += 256) {
            const int r = e / 64, c = e % 64;
            const bool ok = i0 + c < nocc;
            Ca[r][c] = (ok && m0 + r < nao) ? C[(m0 + r) * nocc + i0 + c] : 0.0;
            Cb[r][c] = (ok && n0 + r < nao) ? C[(n0 + r) * nocc + i0 + c] : 0.0;
        }
        __syncthreads();
#pragma unroll 8
        for (int c = 0; c < 64; ++c) s += Ca[ty][c] * Cb[tx][c];
        __syncthreads();
    }
    if (m0 + ty < nao && n0 + tx < nao) D[(m0 + ty) * nao + n0 + tx] = scale * s;
}

__global__ __launch_bounds__(256) void k_density(const double *__restrict__ C, int64_t nao, int32_t nocc,
                                                 double scale, double *__restrict__ D)
{
    density_block(C, nao, nocc, scale, D, blockIdx.x, blockIdx.y);
}

void launch_density(const double *C, int64_t nao, int32_t nocc, double scale, double *D, hipStream_t s)
{
    hipLaunchKernelGGL(k_density, dim3((unsigned)((nao + 15) / 16), (unsigned)((nao + 15) / 16)), dim3(256), 0, s,
                       C, nao, nocc, scale, D);
}

// D = a + b (the open-shell total density).
__global__ void k_add(const double *__restrict__ a, const double *__restrict__ b, int64_t n,
                      double *__restrict__ out)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < n) out[i] = a[i] + b[i];
}

// Rows of B per partial sum of c: about 128 partial sums, 16 to kCSplitRows rows
// each (one workgroup summing 512 rows took 15.6 us of the 82 us build of one
// water), kCSplitRows with the static scratch, which is sized for no more.
static int c_split_rows(int64_t nf_pad, bool fixed)
{
    if (fixed) return kCSplitRows;
    const int64_t r = (nf_pad / 128 + 15) / 16 * 16;
    return (int)std::min<int64_t>(std::max<int64_t>(r, 16), kCSplitRows);
}

// Partial sums of c, block (bx, split) of 512 columns and `rows` rows of B:
// part[split][P] = sum_f d_f B[f][P], the rows' d_f = w_f D[mu_f][nu_f] gathered into
// LDS first.  HBM-bound: B once, 16 bytes a lane.
constexpr int kCCols = 512;
__device__ __forceinline__ void c_partial_block(const double *__restrict__ B, int64_t ld, const double *__restrict__ D,
                                                int64_t nao, const int32_t *__restrict__ fmu,
                                                const int32_t *__restrict__ fnu, const double *__restrict__ fw,
                                                int64_t nf, int64_t nf_pad, int32_t rows, double *__restrict__ part,
                                                unsigned bx, unsigned split)
{
    __shared__ double d[kCSplitRows];
    const int64_t f0 = (int64_t)split * rows;
    const int nr = (int)min((int64_t)rows, nf_pad - f0);
    for (int r = threadIdx.x; r < nr; r += 256) {
        const int64_t f = f0 + r;
        d[r] = f < nf ? fw[f] * D[(int64_t)fmu[f] * nao + fnu[f]] : 0.0;
    }
    __syncthreads();
    const int64_t P = (int64_t)bx * kCCols + 2 * threadIdx.x;
    if (P >= ld) return;
    const double2 *b = reinterpret_cast<const double2 *>(B + f0 * ld + P);
    double2 s0{0.0, 0.0}, s1{0.0, 0.0};
    int r = 0;
#pragma unroll 4
    for (; r + 1 < nr; r += 2) {
        const double2 u = b[r * (ld / 2)], v = b[(r + 1) * (ld / 2)];
        s0.x += d[r] * u.x;
        s0.y += d[r] * u.y;
        s1.x += d[r + 1] * v.x;
        s1.y += d[r + 1] * v.y;
    }
    if (r < nr) {
        const double2 u = b[r * (ld / 2)];
        s0.x += d[r] * u.x;
        s0.y += d[r] * u.y;
    }
    *reinterpret_cast<double2 *>(part + (int64_t)split * ld + P) = double2{s0.x + s1.x, s0.y + s1.y};
}

__global__ __launch_bounds__(256) void k_c_partial(const double *__restrict__ B, int64_t ld,
                                                   const double *__restrict__ D, int64_t nao,
                                                   const int32_t *__restrict__ fmu, const int32_t *__restrict__ fnu,
                                                   const double *__restrict__ fw, int64_t nf, int64_t nf_pad,
                                                   int32_t rows, double *__restrict__ part)
{
    c_partial_block(B, ld, D, nao, fmu, fnu, fw, nf, nf_pad, rows, part, blockIdx.x, blockIdx.y);
}

// c[P] = sum of part[r][P] over the rows, in a fixed order: a workgroup sums 16
// columns, row r in lane group r mod 64, then the groups pairwise.  Workgroups
// past the columns zero J (the pairs that screening dropped keep it).
constexpr int kCSumCols = 16, kCSumGroups = 64, kFillBlock = 8192;
__device__ __forceinline__ void c_sum_block(const double *__restrict__ part, int64_t rows, int64_t ld,
                                            double *__restrict__ c, double *__restrict__ J, int64_t njj, unsigned blk)
{
    __shared__ double red[kCSumGroups][kCSumCols];
    const unsigned ncol = (unsigned)(ld / kCSumCols);
    if (blk >= ncol) {
        const int64_t i0 = (int64_t)(blk - ncol) * kFillBlock;
        for (int64_t i = i0 + threadIdx.x; i < min(i0 + kFillBlock, njj); i += 1024) J[i] = 0.0;
        return;
    }
    const int x = threadIdx.x % kCSumCols, g = threadIdx.x / kCSumCols;
    const int64_t P = (int64_t)blk * kCSumCols + x;
    double s = 0.0;
#pragma unroll 8
    for (int64_t r = g; r < rows; r += kCSumGroups) s += part[r * ld + P];
    red[g][x] = s;
    __syncthreads();
    for (int w = kCSumGroups / 2; w > 0; w >>= 1) {
        if (g < w) red[g][x] += red[g + w][x];
        __syncthreads();
    }
    if (g == 0) c[P] = red[0][x];
}
static unsigned c_sum_blocks(int64_t ld, int64_t njj)
{
    return (unsigned)(ld / kCSumCols + (njj + kFillBlock - 1) / kFillBlock);
}

__global__ __launch_bounds__(1024) void k_c_sum(const double *__restrict__ part, int64_t rows, int64_t ld,
                                                double *__restrict__ c, double *__restrict__ J, int64_t njj)
{
    c_sum_block(part, rows, ld, c, J, njj, blockIdx.x);
}

// J_f = sum_P B[f][P] c_P; one wave per row (ld a multiple of 128: 16-byte loads).
// Diagonal blocks hold both orientations as separate rows, so they write only
// their own element.  HBM-bound: B once.
__device__ __forceinline__ void j_row(const double *__restrict__ B, int64_t ld, const double *__restrict__ c,
                                      const int32_t *__restrict__ fmu, const int32_t *__restrict__ fnu,
                                      const double *__restrict__ fw, int64_t nf, int64_t nao, bool accumulate,
                                      double *__restrict__ J, int64_t f)
{
    const int lane = threadIdx.x & 63;
    if (f >= nf) return;
    const double2 *row = reinterpret_cast<const double2 *>(B + f * ld);
    const double2 *cc = reinterpret_cast<const double2 *>(c);
    double s = 0.0;
#pragma unroll 4
    for (int64_t q = lane; q < ld / 2; q += 64) {
        const double2 b = row[q], v = cc[q];
        s += b.x * v.x;
        s += b.y * v.y;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if (lane == 0) {
        const int64_t mu = fmu[f], nu = fnu[f];
        const double v = accumulate ? J[mu * nao + nu] + s : s;
        J[mu * nao + nu] = v;
        if (fw[f] > 1.5) J[nu * nao + mu] = v;
    }
}

__global__ __launch_bounds__(256) void k_j_rows(const double *__restrict__ B, int64_t ld,
                                                const double *__restrict__ c, const int32_t *__restrict__ fmu,
                                                const int32_t *__restrict__ fnu, const double *__restrict__ fw,
                                                int64_t nf, int64_t nao, int32_t accumulate, double *__restrict__ J)
{
    j_row(B, ld, c, fmu, fnu, fw, nf, nao, accumulate != 0, J, (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6));
}

// ---------------------------------------------------------------------------
// What a build prepares before the half transform, in one launch: the density
// (dmode 1: D = scale C C^T; 2: D copied from the caller's; 0: none) and the
// zero-padded coefficients Cp[nao + 1][ldc] that the half transform reads (C in the
// first ncol columns of the first nao rows).
struct PreArgs {
    const double *C;          // nao x ncol coefficients (the density on the density route)
    double *D, *Cp, *J;       // density, padded coefficients, J
    const int32_t *f_mu, *f_nu;
    const double *f_w, *B;
    double *cpart, *cvec;
    double scale;
    int64_t nao, nf, nf_pad, ld;
    int32_t ncol, ldc, dmode, crows, nsplit_c, pad_;   // crows: rows of B per partial sum of c
};
constexpr int kPadBlock = 1024;   // elements of Cp (or of a copied D) per workgroup

static unsigned density_blocks(const PreArgs &a)
{
    const int64_t g = (a.nao + 15) / 16;
    return (unsigned)(a.dmode == 1 ? g * g : a.dmode == 2 ? (a.nao * a.nao + kPadBlock - 1) / kPadBlock : 0);
}
static unsigned prep_blocks(const PreArgs &a)
{
    return density_blocks(a) + (unsigned)(((a.nao + 1) * a.ldc + kPadBlock - 1) / kPadBlock);
}

__device__ __forceinline__ void prep_block(const PreArgs &a, unsigned local, unsigned nd)
{
    if (local < nd) {
        if (a.dmode == 1) {
            const unsigned gx = (unsigned)((a.nao + 15) / 16);
            density_block(a.C, a.nao, a.ncol, a.scale, a.D, local % gx, local / gx);
        } else {
            const int64_t i0 = (int64_t)local * kPadBlock;
            for (int64_t i = i0 + threadIdx.x; i < min(i0 + kPadBlock, a.nao * a.nao); i += 256) a.D[i] = a.C[i];
        }
        return;
    }
    const int64_t i0 = (int64_t)(local - nd) * kPadBlock, n = (a.nao + 1) * a.ldc;
    for (int64_t i = i0 + threadIdx.x; i < min(i0 + kPadBlock, n); i += 256) {
        const int64_t r = i / a.ldc, c = i % a.ldc;
        a.Cp[i] = (r < a.nao && c < a.ncol) ? a.C[r * a.ncol + c] : 0.0;
    }
}

__global__ __launch_bounds__(256) void k_prep(PreArgs a, unsigned nd)
{
    prep_block(a, blockIdx.x, nd);
}

// The steps around the half transform for the molecules of a batch in shared
// launches, one per step: workgroup b of a step belongs to molecule m for
// blk_start[m] <= b < blk_start[m + 1] and runs what block b - blk_start[m] of that
// molecule's own launch runs, with the same arithmetic per element, so J and c are
// bitwise those of separate builds.
constexpr int kPreGroupMax = 16;
struct PreGroup {
    int32_t n;
    uint32_t blk_start[kPreGroupMax + 1];
    uint32_t nd[kPreGroupMax];
    PreArgs a[kPreGroupMax];
};
static_assert(sizeof(PreGroup) <= 4096, "kernel arguments are limited to 4 KB");
enum { PRE_PREP, PRE_CPART, PRE_CSUM, PRE_JROWS };

__device__ __forceinline__ int pre_member(const PreGroup &g, unsigned &local)
{
    int m = 0;
    while (m + 1 < g.n && blockIdx.x >= g.blk_start[m + 1]) ++m;
    local = blockIdx.x - g.blk_start[m];
    return m;
}

__global__ __launch_bounds__(256) void k_prep_group(PreGroup g)
{
    unsigned local;
    const int m = pre_member(g, local);
    prep_block(g.a[m], local, g.nd[m]);
}

__global__ __launch_bounds__(256) void k_c_partial_group(PreGroup g)
{
    unsigned local;
    const PreArgs &a = g.a[pre_member(g, local)];
    const unsigned gx = (unsigned)((a.ld + kCCols - 1) / kCCols);
    c_partial_block(a.B, a.ld, a.D, a.nao, a.f_mu, a.f_nu, a.f_w, a.nf, a.nf_pad, a.crows, a.cpart, local % gx,
                    local / gx);
}

__global__ __launch_bounds__(1024) void k_c_sum_group(PreGroup g)
{
    unsigned local;
    const PreArgs &a = g.a[pre_member(g, local)];
    c_sum_block(a.cpart, a.nsplit_c, a.ld, a.cvec, a.J, a.nao * a.nao, local);
}

__global__ __launch_bounds__(256) void k_j_rows_group(PreGroup g)
{
    unsigned local;
    const PreArgs &a = g.a[pre_member(g, local)];
    j_row(a.B, a.ld, a.cvec, a.f_mu, a.f_nu, a.f_w, a.nf, a.nao, false, a.J, (int64_t)local * 4 + (threadIdx.x >> 6));
}

// One step as shared launches of up to kPreGroupMax molecules.
static void launch_pre_group(int st, const std::vector<PreArgs> &as, hipStream_t s)
{
    for (size_t first = 0; first < as.size(); first += kPreGroupMax) {
        PreGroup g{};
        int64_t total = 0;
        for (size_t i = first; i < as.size() && g.n < kPreGroupMax; ++i) {
            const PreArgs &a = as[i];
            g.blk_start[g.n] = (uint32_t)total;
            g.nd[g.n] = density_blocks(a);
            g.a[g.n++] = a;
            total += st == PRE_PREP    ? prep_blocks(a)
                     : st == PRE_CPART ? (a.ld + kCCols - 1) / kCCols * a.nsplit_c
                     : st == PRE_CSUM  ? c_sum_blocks(a.ld, a.nao * a.nao)
                                       : (a.nf + 3) / 4;
        }
        g.blk_start[g.n] = (uint32_t)total;
        if (total <= 0) continue;
        const dim3 grid((unsigned)total);
        switch (st) {
        case PRE_PREP: hipLaunchKernelGGL(k_prep_group, grid, dim3(256), 0, s, g); break;
        case PRE_CPART: hipLaunchKernelGGL(k_c_partial_group, grid, dim3(256), 0, s, g); break;
        case PRE_CSUM: hipLaunchKernelGGL(k_c_sum_group, grid, dim3(1024), 0, s, g); break;
        default: hipLaunchKernelGGL(k_j_rows_group, grid, dim3(256), 0, s, g); break;
        }
    }
}

// ---------------------------------------------------------------------------
// Half transform.  MFMA operands: A = B[row_k][P] (lane: P = l%16,
// k = l/16), B = Cs[k][i] (lane: k = l/16, i = l%16); accumulator r holds
// row P = l/16 + 4r.

enum { OUT_F64 = 0, OUT_F32 = 1, OUT_BF16X2 = 2, OUT_I8 = 3 };
typedef double f64x2 __attribute__((ext_vector_type(2)));

struct HTArgs {
    const double *B;          // [f][ld]
    int64_t ld;               // naux_pad
    const double *C;          // [nao + 1][ldc]: coefficients zero-padded to ldc columns, row nao zero
    int32_t ncol;             // columns of the coefficients
    int32_t ldc;
    const int32_t *hk_off, *hk_row, *hk_nu;   // partner lists, each padded to a multiple of kHtChunk
    void *X;                  // [nao][plen][ncol]: aux rows p_begin .. p_begin + plen - 1
                              // (int8 slices: [nao][kdim/64][nslice][64])
    void *Xlo;                // second plane for the BF16 split; block scales for int8
    int64_t p_begin, plen;    // aux slab (multiples of 128)
    const int32_t *order;     // blockIdx.y -> AO function (longest list first)
    int32_t nslice;           // int8 slices stored
};


__device__ __forceinline__ unsigned short f32_to_bf16_rne(float x)
{
    unsigned int u = __float_as_uint(x);
    const unsigned int rounding = 0x7fffu + ((u >> 16) & 1u);
    return (unsigned short)((u + rounding) >> 16);
}
__device__ __forceinline__ float bf16_to_f32(unsigned short h) { return __uint_as_float(((unsigned int)h) << 16); }

// LDS of one k chunk of the half transform: kHtChunk rows of the 128-wide B
// tile (the MFMA A operand, LDA apart), then kHtChunk rows of the pass's NCOL
// coefficient columns (LDC apart).  The row pitches put the four k rows that
// one fragment read touches on alternating halves of the banks.
template <int NCOL> struct HtLds {
    static constexpr int PAD = (16 - NCOL % 32 + 32) % 32;
    static constexpr int LDC = NCOL + PAD;
    static constexpr int LDA = 128 + 16;
    static constexpr int DOUBLES = kHtChunk * (LDA + LDC);
};

// Int8 output of one half-transform workgroup (mu, 128 aux rows p0.., the
// column pass ic0.. of width w = min(NCOL, ncol - ic0), stored w_e = w
// rounded up to even wide).  Contraction index inside the slab:
//   k = plen * ic0 + (P - p_begin) * w_e + (col - ic0),
// so the workgroup owns 128 w_e / 256 whole scale blocks and one contiguous
// byte range of the row (chunks of 64 k, nslice slices each).  Per block: the
// largest |x| (LDS atomics on the bit pattern, which orders like the value
// for non-negative doubles), e = the least exponent with 2^e > |x|max
// 128/127, the scale 2^e to g.Xlo; then x 2^-e = sum_s a_s 2^{-7(s+1)} by
// repeated rounding, every step exact in FP64 (a_0 = rint(128 x 2^-e) in
// [-127, 127], later a_s in [-64, 64]); slices 0 .. nslice - 1 are stored
// (four for int8_fast, whose K never reads a_4).  The pad column stores zeros.
// Slicing runs from LDS, 32 aux rows at a time: the two waves that hold them
// write their FP64 values to the first operand buffer in k order, then every
// thread slices four consecutive k and stores one 4-byte word per slice, so
// the registers of the accumulators are the only large live state.  The
// block maxima and exponents sit at the end of the second buffer.
template <int NIB>
__device__ __forceinline__ void store_i8(const HTArgs &g, const f64x4 (&acc)[NIB], double *st,
                                         unsigned char *tab, int mu, int64_t p0, int ic0, int tid, int lane,
                                         int wave, int kl)
{
    constexpr int NCOL = NIB * 16;
    static_assert(32 * NCOL * 8 <= HtLds<NCOL>::DOUBLES * 8, "32 rows of FP64 must fit a buffer");
    static_assert(128 * 12 <= HtLds<NCOL>::DOUBLES * 8, "block tables must fit a buffer");
    unsigned long long *bmax = reinterpret_cast<unsigned long long *>(tab);
    int *bexp = reinterpret_cast<int *>(tab + 128 * 8);
    const int w = min(NCOL, g.ncol - ic0), we = w + (w & 1);
    const int64_t kbase = g.plen * ic0 + (p0 - g.p_begin) * we;     // a multiple of kI8Block
    const int64_t kdim = g.plen * (int64_t)(g.ncol + (g.ncol & 1));
    const int64_t nblk = kdim / kI8Block;
    __syncthreads();   // the k loop's LDS reads are done
    if (tid < 128) bmax[tid] = 0ull;
    __syncthreads();
    // Block maxima.  A lane's values of one r lie in one aux row, whose we <=
    // 160 k span at most two blocks (lo, hi); the 16 lanes of that row (one
    // DPP row, lane & 15) reduce both by butterfly, then one lane of each row
    // updates the two blocks' maxima in LDS.
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int row0 = (16 * wave + kl + 4 * r) * we;
        const int blo = row0 / kI8Block;
        double mlo = 0.0, mhi = 0.0;
#pragma unroll
        for (int j = 0; j < NIB; ++j) {
            const int c = j * 16 + (lane & 15);
            const double v = c < w ? fabs(acc[j][r]) : 0.0;
            if ((row0 + c) / kI8Block == blo) mlo = fmax(mlo, v);
            else mhi = fmax(mhi, v);
        }
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) {
            mlo = fmax(mlo, __shfl_xor(mlo, o, 16));
            mhi = fmax(mhi, __shfl_xor(mhi, o, 16));
        }
        if ((lane & 15) == 0) {
            atomicMax(&bmax[blo], (unsigned long long)__double_as_longlong(mlo));
            if ((row0 + we - 1) / kI8Block != blo)
                atomicMax(&bmax[blo + 1], (unsigned long long)__double_as_longlong(mhi));
        }
    }
    __syncthreads();
    const int nb = 128 * we / kI8Block;
    if (tid < nb) {
        const double m = __longlong_as_double((long long)bmax[tid]);
        const int e = m > 0.0 ? ilogb(m * (128.0 / 127.0)) + 1 : 0;
        bexp[tid] = e;
        static_cast<double *>(g.Xlo)[(int64_t)mu * nblk + kbase / kI8Block + tid] = ldexp(1.0, e);
    }
    unsigned char *dst = static_cast<unsigned char *>(g.X) + (int64_t)mu * kdim * g.nslice +
                         (kbase / kI8Chunk) * (kI8Chunk * g.nslice);
    const int qk = 32 * we;                                            // k of 32 aux rows
    for (int q = 0; q < 4; ++q) {
        __syncthreads();   // exponents written; the previous quarter's values read
        if ((wave >> 1) == q) {
#pragma unroll
            for (int j = 0; j < NIB; ++j) {
                const int c = j * 16 + (lane & 15);
                if (c >= we) continue;
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    st[(16 * (wave & 1) + kl + 4 * r) * we + c] = c < w ? acc[j][r] : 0.0;
            }
        }
        __syncthreads();
        for (int it = tid; it < qk / 4; it += 512) {
            const int kq = 4 * it, k = q * qk + kq;                  // k within the workgroup's range
            const int e = bexp[k / kI8Block];                        // four k share a block
            double t[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) t[u] = ldexp(st[kq + u], -e);
            unsigned char *d = dst + (k / kI8Chunk) * (kI8Chunk * g.nslice) + (k % kI8Chunk);
#pragma unroll
            for (int sl = 0; sl < kI8Slices; ++sl) {
                if (sl >= g.nslice) break;
                unsigned int word = 0;
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    t[u] *= 128.0;
                    const double a = rint(t[u]);
                    t[u] -= a;
                    word |= (unsigned int)(unsigned char)(signed char)(int)a << (8 * u);
                }
                *reinterpret_cast<unsigned int *>(d + sl * kI8Chunk) = word;
            }
        }
    }
}

// s_waitcnt immediate for vmcnt(0) (gfx9 encoding; expcnt and lgkmcnt at
// their maxima do not wait), issued through the builtin so the compiler's own
// wait insertion knows the loads have retired.
constexpr int kHtWaitVm0 = 0 | (7 << 4) | (15 << 8);

// Workgroup (mu, 128-row P tile, column pass of NIB*16 columns) of eight
// waves, each 16 aux rows x NIB fragments: X[mu][P][i] = sum over mu's
// partners k of B[row_k][P] C[nu_k][i].  The partners run in chunks of
// kHtChunk; each chunk's B rows (1 KB each) and coefficient rows move from
// global memory straight into one of two LDS buffers (global_load_lds, 16
// bytes a lane, no registers), the next chunk in flight while the MFMAs use
// the current one, one barrier per chunk.  Wave w brings rows 2w and 2w+1 of
// both operands; the partner indices of the chunk after next are loaded
// into a register (lane l: entry l of the chunk) with the DMA, so issuing a
// chunk never waits on an index load.  The padded partner lists make every
// chunk whole; the padded coefficients keep every 16-byte piece in bounds.
template <int OUT, int NIB>
__device__ __forceinline__ void halftrans_tile(HTArgs g, unsigned bx, unsigned by, unsigned bz)
{
    constexpr int KC = kHtChunk, NCOL = NIB * 16;
    constexpr int LDA = HtLds<NCOL>::LDA, LDC = HtLds<NCOL>::LDC;
    constexpr int NPR = (NCOL + 127) / 128;             // DMA instructions per coefficient row
    // two chunk buffers as separate arrays: the compiler then tells a read of
    // one from a DMA into the other and does not wait for unrelated loads
    __shared__ __attribute__((aligned(1024))) double sb0[HtLds<NCOL>::DOUBLES];
    __shared__ __attribute__((aligned(1024))) double sb1[HtLds<NCOL>::DOUBLES];
    const int mu = g.order[by];
    const int64_t p0 = g.p_begin + (int64_t)bx * 128;
    const int ic0 = bz * NCOL;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kb = g.hk_off[mu], ke = g.hk_off[mu + 1];
    const int nch = (ke - kb) / KC;
    const int kl = lane >> 4;   // k within an MFMA step

    f64x4 acc[NIB];
#pragma unroll
    for (int j = 0; j < NIB; ++j) acc[j] = f64x4{0.0, 0.0, 0.0, 0.0};

    // partner indices of chunk ci (lane l: entry l % 16; past the list: its last entry)
    int rowv = 0, nuv = 0;
    auto load_idx = [&](int ci) {
        const int k = min(kb + ci * KC + (lane & 15), ke - 1);
        rowv = g.hk_row[k];
        nuv = g.hk_nu[k];
    };
    auto dma = [&](double *buf) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int r = 2 * wave + i;
            const int row = __builtin_amdgcn_readlane(rowv, r);
            const int nu = __builtin_amdgcn_readlane(nuv, r);
            __builtin_amdgcn_global_load_lds(
                (const void *)(g.B + (int64_t)row * g.ld + p0 + 2 * lane),
                (__attribute__((address_space(3))) void *)(buf + r * LDA), 16, 0, 0);
#pragma unroll
            for (int q = 0; q < NPR; ++q)
                if (q * 128 + 2 * lane < NCOL)
                    __builtin_amdgcn_global_load_lds(
                        (const void *)(g.C + (int64_t)nu * g.ldc + ic0 + q * 128 + 2 * lane),
                        (__attribute__((address_space(3))) void *)(buf + KC * LDA + r * LDC + q * 128), 16, 0, 0);
        }
    };
    // one chunk: wait for its DMA (every wave's, through the barrier, which
    // also tells that every wave has finished reading `nxt`), start the next
    // chunk's DMA into `nxt`, then the MFMAs on `cur`
    auto step = [&](const double *cur, double *nxt, int c) {
        __builtin_amdgcn_s_waitcnt(kHtWaitVm0);
        __syncthreads();
        if (c + 1 < nch) {
            dma(nxt);
            load_idx(c + 2);
        }
        __builtin_amdgcn_sched_barrier(0);
        const double *as = cur + kl * LDA + 16 * wave + (lane & 15);
        const double *cs = cur + KC * LDA + kl * LDC + (lane & 15);
#pragma unroll
        for (int ks = 0; ks < KC / 4; ++ks) {
            const double a = as[ks * 4 * LDA];
#pragma unroll
            for (int j = 0; j < NIB; ++j)
                acc[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, cs[ks * 4 * LDC + j * 16], acc[j], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };

    if (nch > 0) {
        load_idx(0);
        dma(sb0);
        load_idx(1);
        for (int c = 0; c < nch; c += 2) {
            step(sb0, sb1, c);
            if (c + 1 < nch) step(sb1, sb0, c + 1);
        }
    }

    if constexpr (OUT == OUT_I8) {
        store_i8(g, acc, sb0, reinterpret_cast<unsigned char *>(sb1), mu, p0, ic0, tid, lane, wave, kl);
        return;
    }
#pragma unroll
    for (int j = 0; j < NIB; ++j) {
        const int col = ic0 + j * 16 + (lane & 15);
        if (col >= g.ncol) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int64_t P = p0 + 16 * wave + kl + 4 * r;
            const int64_t o = ((int64_t)mu * g.plen + (P - g.p_begin)) * g.ncol + col;
            const double v64 = acc[j][r];
            if (OUT == OUT_F64) {
                __builtin_nontemporal_store(v64, static_cast<double *>(g.X) + o);
            } else if (OUT == OUT_F32) {
                const int64_t k = (P - g.p_begin) * g.ncol + col;
                static_cast<float *>(g.X)[(int64_t)mu * g.plen * g.ncol + f32_k_slot(k)] = (float)v64;
            } else {
                const float v = (float)v64;
                const unsigned short hi = f32_to_bf16_rne(v);
                const unsigned short lo = f32_to_bf16_rne(v - bf16_to_f32(hi));
                static_cast<unsigned short *>(g.X)[o] = hi;
                static_cast<unsigned short *>(g.Xlo)[o] = lo;
            }
        }
    }
}

template <int OUT, int NIB>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4, 4)))
void k_halftrans(HTArgs g)
{
    halftrans_tile<OUT, NIB>(g, blockIdx.x, blockIdx.y, blockIdx.z);
}

// Half transforms of several molecules (the same output and fragment count)
// in one launch: workgroup b runs workgroup b - blk_start[m] of molecule m's own
// grid (gx P tiles fastest, then gy AO functions, then column passes), with
// its arguments passed by value, so small molecules share the chip.
constexpr int kHtGroupMax = 16;
struct HtGroup {
    int32_t n;
    uint32_t blk_start[kHtGroupMax + 1];
    uint32_t gx[kHtGroupMax], gy[kHtGroupMax];
    HTArgs g[kHtGroupMax];
};
static_assert(sizeof(HtGroup) <= 4096, "kernel arguments are limited to 4 KB");

template <int OUT, int NIB>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4, 4)))
void k_halftrans_group(HtGroup grp)
{
    int m = 0;
    while (m + 1 < grp.n && blockIdx.x >= grp.blk_start[m + 1]) ++m;
    const unsigned local = blockIdx.x - grp.blk_start[m];
    const unsigned bx = local % grp.gx[m], rest = local / grp.gx[m];
    halftrans_tile<OUT, NIB>(grp.g[m], bx, rest % grp.gy[m], rest / grp.gy[m]);
}

// Coefficients for the half transform: Cp[nao + 1][ldc] with C in the first
// ncol columns of the first nao rows and zeros elsewhere.
__global__ __launch_bounds__(256) void k_pad_coef(const double *__restrict__ C, int64_t nao, int32_t ncol,
                                                  int32_t ldc, double *__restrict__ Cp)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= (nao + 1) * ldc) return;
    const int64_t r = i / ldc, c = i % ldc;
    Cp[i] = (r < nao && c < ncol) ? C[r * ncol + c] : 0.0;
}

template <int OUT>
static void launch_halftrans(const HTArgs &h, int64_t nao, hipStream_t s)
{
    const int nib = ht_pass_frags(h.ncol);
    dim3 grid((unsigned)(h.plen / 128), (unsigned)nao, (unsigned)ht_passes(h.ncol));
#define HT_CASE(N) \
    case N: hipLaunchKernelGGL((k_halftrans<OUT, N>), grid, dim3(512), 0, s, h); break;
    switch (nib) {
        HT_CASE(1) HT_CASE(2) HT_CASE(3) HT_CASE(4) HT_CASE(5) HT_CASE(6) HT_CASE(7) HT_CASE(8)
        HT_CASE(9) HT_CASE(10)
    }
#undef HT_CASE
}
static_assert(kHtMaxFrag == 10, "launch_halftrans instantiates 1..kHtMaxFrag fragments");

// Half transforms of several molecules with output OUT (FP64 or int8
// slices): those with the same fragment count share launches of
// k_halftrans_group (up to kHtGroupMax each).
template <int OUT>
static void launch_halftrans_groups(const std::vector<std::pair<HTArgs, int64_t>> &hs, hipStream_t s)
{
    for (int nib = 1; nib <= kHtMaxFrag; ++nib) {
        HtGroup grp{};
        int64_t total = 0;
        auto flush = [&]() {
            if (grp.n == 0) return;
            grp.blk_start[grp.n] = (uint32_t)total;
#define HT_CASE(N) \
    case N: hipLaunchKernelGGL((k_halftrans_group<OUT, N>), dim3((unsigned)total), dim3(512), 0, s, grp); break;
            switch (nib) {
                HT_CASE(1) HT_CASE(2) HT_CASE(3) HT_CASE(4) HT_CASE(5) HT_CASE(6) HT_CASE(7) HT_CASE(8)
                HT_CASE(9) HT_CASE(10)
            }
#undef HT_CASE
            grp = HtGroup{};
            total = 0;
        };
        for (const auto &e : hs) {
            const HTArgs &h = e.first;
            if (ht_pass_frags(h.ncol) != nib) continue;
            const int64_t gx = h.plen / 128, gy = e.second, gz = ht_passes(h.ncol);
            const int64_t nb = gx * gy * gz;
            if (nb <= 0) continue;
            if (grp.n == kHtGroupMax || total + nb > (int64_t)UINT32_MAX / 2) flush();
            grp.blk_start[grp.n] = (uint32_t)total;
            grp.gx[grp.n] = (uint32_t)gx;
            grp.gy[grp.n] = (uint32_t)gy;
            grp.g[grp.n++] = h;
            total += nb;
        }
        flush();
    }
}

static void dispatch_halftrans(int precision, const HTArgs &h, int64_t nao, hipStream_t s)
{
    switch (precision) {
    case DFJK_FP64: launch_halftrans<OUT_F64>(h, nao, s); break;
    case DFJK_MIXED_FP32: launch_halftrans<OUT_F32>(h, nao, s); break;
    case DFJK_MIXED_BF16X3: launch_halftrans<OUT_BF16X2>(h, nao, s); break;
    default: launch_halftrans<OUT_I8>(h, nao, s); break;
    }
}

// Dense expansion for the D route: Bt[mu][P][nu] = B[f(mu,nu)][P] (0 elsewhere).
// Workgroup (32 aux rows, mu): 64 nu at a time through LDS, so that B is read along
// P (256 bytes a row) and Bt written along nu (512 bytes a row); the partner list is
// sorted by nu.  Bound by the write of Bt (7 waters, 226 MB: one thread per P and a
// strided store per nu took 270-310 us).
constexpr int kExpP = 32, kExpN = 64;
__global__ __launch_bounds__(256) void k_expand_B(const double *__restrict__ B, int64_t ld,
                                                  const int32_t *__restrict__ hk_off,
                                                  const int32_t *__restrict__ hk_row,
                                                  const int32_t *__restrict__ hk_nu, int64_t nao,
                                                  int64_t p_begin, int64_t plen, double *__restrict__ Bt)
{
    __shared__ double tile[kExpN][kExpP + 1];
    const int mu = blockIdx.y, tid = threadIdx.x;
    const int64_t pl0 = (int64_t)blockIdx.x * kExpP;   // plen is a multiple of 128
    const int px = tid % kExpP, kx = tid / kExpP, nx = tid % kExpN, py = tid / kExpN;
    const double *src = B + p_begin + pl0 + px;
    double *dst = Bt + ((int64_t)mu * plen + pl0) * nao;
    int k = hk_off[mu];
    const int ke = hk_off[mu + 1];
    for (int64_t n0 = 0; n0 < nao; n0 += kExpN) {
        for (int i = kx; i < kExpN; i += 256 / kExpP) tile[i][px] = 0.0;
        __syncthreads();
        // entries k .. of this chunk: at most kExpN of them (each nu once; padding
        // entries name row nao, past every chunk)
        int used = 0;
        for (int i = kx; i < kExpN && k + i < ke; i += 256 / kExpP) {
            const int64_t nu = hk_nu[k + i];
            if (nu < n0 + kExpN && nu < nao) tile[nu - n0][px] = src[(int64_t)hk_row[k + i] * ld];
        }
        for (int i = 0; i < kExpN && k + i < ke && hk_nu[k + i] < n0 + kExpN; ++i) ++used;
        k += used;
        __syncthreads();
        if (n0 + nx < nao)
            for (int r = py; r < kExpP; r += 256 / kExpN) dst[(int64_t)r * nao + n0 + nx] = tile[nx][r];
        __syncthreads();
    }
}

// [U | W] = [C + C0 | C - C0] (nao x 2 nocc): 2(C C^T - C0 C0^T) = U W^T + W U^T.
__global__ void k_uw(const double *__restrict__ C, const double *__restrict__ C0, int64_t nao, int32_t nocc,
                     double *__restrict__ U, double *__restrict__ W)
{
    const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (e >= nao * nocc) return;
    const double c = C[e], c0 = C0[e];
    U[e] = c + c0;
    W[e] = c - c0;
}

// Incremental K: K = K0 + G + G^T with G = X_U X_W^T held as split-K partial
// tiles over every 128x128 tile (rectangular order t = tm + tn * ntm).  One
// block per lower tile and 16-row chunk sums both G[m][n] and G[n][m] in a
// fixed order, writes K symmetric, and sums D o K for E_K.
__global__ __launch_bounds__(256) void k_k_reduce_delta(const double *__restrict__ part, int nsplit, int ntm,
                                                        int64_t nao, const double *__restrict__ K0,
                                                        const double *__restrict__ D, double *__restrict__ K,
                                                        double *__restrict__ Epart)
{
    __shared__ double red[256];
    const int t = blockIdx.x;
    int tm = (int)((sqrt(8.0 * (double)t + 1.0) - 1.0) * 0.5);
    while (tm * (tm + 1) / 2 > t) --tm;
    while ((tm + 1) * (tm + 2) / 2 <= t) ++tm;
    const int tn = t - tm * (tm + 1) / 2;
    const int64_t tile_mn = tm + (int64_t)tn * ntm, tile_nm = tn + (int64_t)tm * ntm;
    const int64_t nt = (int64_t)ntm * ntm, TT = (int64_t)kTileK * kTileK;
    const int chunk = blockIdx.y;
    double e = 0.0;
    for (int q = threadIdx.x; q < 16 * kTileK; q += 256) {
        const int row = chunk * 16 + q / kTileK, col = q % kTileK;
        const int64_t m = (int64_t)tm * kTileK + row, n = (int64_t)tn * kTileK + col;
        if (m >= nao || n >= nao || n > m) continue;
        double g1 = 0.0, g2 = 0.0;
#pragma unroll 8
        for (int sp = 0; sp < nsplit; ++sp) {
            g1 += part[(sp * nt + tile_mn) * TT + row * kTileK + col];
            g2 += part[(sp * nt + tile_nm) * TT + col * kTileK + row];
        }
        const double v = K0[m * nao + n] + (g1 + g2);
        K[m * nao + n] = v;
        double w = 1.0;
        if (m != n) {
            K[n * nao + m] = v;
            w = 2.0;
        }
        e += w * D[m * nao + n] * v;
    }
    red[threadIdx.x] = e;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) Epart[(int64_t)t * gridDim.y + chunk] = red[0];
}

// ---------------------------------------------------------------------------
// Split-K reduction of the K tiles: K[m][n] = scale * sum_s partial[s][t][..]
// in a fixed order, mirrored for off-diagonal tiles, plus per-block partial
// sums of D[m][n] K[m][n] (weight 2 off the diagonal tiles) for E_K.
// Rows of a tile per reduction workgroup: small enough that the grid has
// many workgroups (each lane sums its splits in turn, so the loads of many
// lanes in flight hide their latency).
constexpr int kReduceRows = 4;
constexpr int reduce_chunks(int T) { return T / kReduceRows; }

__device__ __forceinline__ void reduce_tile(const double *__restrict__ part, int nsplit, int ntm, int T, int64_t nao,
                                            double scale, const double *__restrict__ D, double *__restrict__ K,
                                            double *__restrict__ Epart, const int t, const int chunk)
{
    __shared__ double red[256];
    const int ntiles = ntm * (ntm + 1) / 2;
    int tm = (int)((sqrt(8.0 * (double)t + 1.0) - 1.0) * 0.5);
    while (tm * (tm + 1) / 2 > t) --tm;
    while ((tm + 1) * (tm + 2) / 2 <= t) ++tm;
    const int tn = t - tm * (tm + 1) / 2;
    double e = 0.0;
    for (int q = threadIdx.x; q < kReduceRows * T; q += 256) {
        const int row = chunk * kReduceRows + q / T, col = q % T;
        const int64_t m = (int64_t)tm * T + row, n = (int64_t)tn * T + col;
        // the upper half of a diagonal tile is mirrored from its lower half
        if (m >= nao || n >= nao || n > m) continue;
        const int64_t off = (int64_t)t * T * T + row * T + col;
        double s = 0.0;
#pragma unroll 8
        for (int sp = 0; sp < nsplit; ++sp) s += part[(int64_t)sp * ntiles * T * T + off];
        s *= scale;
        K[m * nao + n] = s;
        double w = 1.0;
        if (m != n) {
            K[n * nao + m] = s;
            w = 2.0;
        }
        e += w * D[m * nao + n] * s;
    }
    red[threadIdx.x] = e;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) Epart[(int64_t)t * reduce_chunks(T) + chunk] = red[0];
}

// block (t, chunk): lower tile t (T wide), rows kReduceRows chunk onwards
__global__ __launch_bounds__(256) void k_k_reduce(const double *__restrict__ part, int nsplit, int ntm, int T,
                                                  int64_t nao, double scale, const double *__restrict__ D,
                                                  double *__restrict__ K, double *__restrict__ Epart)
{
    reduce_tile(part, nsplit, ntm, T, nao, scale, D, K, Epart, blockIdx.x, blockIdx.y);
}

// Grouped reduction for a batch: blocks blk_start[p] .. blk_start[p+1]-1 reduce
// molecule p, whose tiles are T[p] wide; the grid has reduce_chunks(kTileK)
// chunks in y (the most any width needs) and molecule p uses the first
// reduce_chunks(T[p]).  Descriptors by value.
constexpr int kReduceGroupMax = 16;
struct ReduceGroup {
    int32_t n;
    int32_t blk_start[kReduceGroupMax + 1];
    int32_t nsplit[kReduceGroupMax], ntm[kReduceGroupMax], T[kReduceGroupMax];
    int64_t nao[kReduceGroupMax];
    const double *part[kReduceGroupMax], *D[kReduceGroupMax];
    double *K[kReduceGroupMax], *Epart[kReduceGroupMax];
};

__global__ __launch_bounds__(256) void k_k_reduce_grouped(ReduceGroup grp, double scale)
{
    const int b = blockIdx.x;
    int p = 0;
    while (p + 1 < grp.n && b >= grp.blk_start[p + 1]) ++p;
    if ((int)blockIdx.y >= reduce_chunks(grp.T[p])) return;   // past this molecule's rows
    reduce_tile(grp.part[p], grp.nsplit[p], grp.ntm[p], grp.T[p], grp.nao[p], scale, grp.D[p], grp.K[p],
                grp.Epart[p], b - grp.blk_start[p], blockIdx.y);
}

__device__ __forceinline__ void energies_body(const double *__restrict__ c, int64_t naux,
                                              const double *__restrict__ Epart, int64_t nEpart, double fk,
                                              double *__restrict__ E)
{
    __shared__ double r1[256], r2[256];
    double a = 0.0, b = 0.0;
    for (int64_t i = threadIdx.x; i < naux; i += 256) a += c[i] * c[i];
    for (int64_t i = threadIdx.x; i < nEpart; i += 256) b += Epart[i];
    r1[threadIdx.x] = a;
    r2[threadIdx.x] = b;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) {
            r1[threadIdx.x] += r1[threadIdx.x + w];
            r2[threadIdx.x] += r2[threadIdx.x + w];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        E[0] = 0.5 * r1[0];
        E[1] = fk * r2[0];
    }
}

__global__ __launch_bounds__(256) void k_energies(const double *__restrict__ c, int64_t naux,
                                                  const double *__restrict__ Epart, int64_t nEpart, double fk,
                                                  double *__restrict__ E)
{
    energies_body(c, naux, Epart, nEpart, fk, E);
}

// one block per molecule of a batch
constexpr int kEnergyGroupMax = 64;
struct EnergyGroup {
    const double *c[kEnergyGroupMax], *Epart[kEnergyGroupMax];
    int64_t naux[kEnergyGroupMax], nEpart[kEnergyGroupMax];
    double *E[kEnergyGroupMax];
};

__global__ __launch_bounds__(256) void k_energies_grouped(EnergyGroup grp, double fk)
{
    const int p = blockIdx.x;
    energies_body(grp.c[p], grp.naux[p], grp.Epart[p], grp.nEpart[p], fk, grp.E[p]);
}

// ---------------------------------------------------------------------------

// Split-K count for the K contraction: the largest count whose workgroups
// (per_cu per CU) fit in one round, so no nearly empty last round idles the
// chip; at least 256 k values per split.  short_k: 512 where that still gives eight
// workgroups per CU (390 AO x 74,880 k, 144 / 288 splits: 0.279 / 0.282 ms, and the
// reduction reads half the partial tiles: 39 -> 20 us), 128 where 256 leaves fewer
// than four (30 AO x 640 k, 2 / 5 splits: 15.8 / 7.9 us).  The increment takes no
// splits below 256 k: its reduction reads both triangles of every split, one of them
// across rows (whole increments of 150 / 210 AO with and without: 0.72 and 0.63, 1.44 and
// 1.12 ms; the split of 480 AO at 512 k gains, 4.41 -> 4.13).
int mixed_nsplit(int64_t nao, int64_t kdim, bool lower, int num_cus);
int i8_fast_tile(int64_t nao);
int i8_nsplit(int64_t nao, int64_t kdim, bool lower, int tile, int num_cus);
void launch_gemm_i8(bool lower, const void *A, const double *sA, const void *B, const double *sB, int64_t nao,
                    int64_t kdim, int nsplit, bool fast, int tile, double *part, hipStream_t s);
void launch_gemm_i8_group(bool fast, int tile, int n, const void *const *X, const double *const *sX,
                          const int64_t *nao, const int64_t *kdim, const int *nsplit, double *const *part,
                          hipStream_t s);

static int choose_ksplit(int ntiles, int64_t kdim, int num_cus, int per_cu, bool short_k, bool delta)
{
    const int slots = per_cu * (num_cus > 0 ? num_cus : 256);
    int ns = ntiles >= slots ? 1 : slots / ntiles;
    const int64_t cus = num_cus > 0 ? num_cus : 256;
    int64_t maxs = kdim / 256;
    if (short_k) {
        if (ntiles * (kdim / 512) >= 8 * cus) maxs = kdim / 512;
        else if (!delta) maxs = std::max<int64_t>(maxs, std::min<int64_t>(kdim / 128, 4 * cus / ntiles));
    }
    if (ns > maxs) ns = (int)(maxs > 0 ? maxs : 1);
    if (ns < 1) ns = 1;
    return ns;
}

// Parts of each of `ranges` k ranges of the FP32 syrk: as many as asked for, each of whole
// folds (512 k), none empty (24 waters: 9 parts asked of 10,880 k are 8 of 1,536; the
// ninth was 24 of 216 splits of zeros, written and read back).
static int f32_parts(int64_t kdim, int ranges, int64_t want)
{
    const int64_t len = (kdim + ranges - 1) / ranges, n = std::max<int64_t>(1, want);
    const int64_t part = (int64_t)align_up((size_t)((len + n - 1) / n), 512);
    return (int)((len + part - 1) / part);
}

static int xcd_round(int ns) { return ns >= kXcds ? ns / kXcds * kXcds : ns; }

BuildLayout build_layout(const Plan &p, int32_t nocc, int32_t precision, bool with_D, bool delta, int nsplit,
                         bool allow_overlap, int64_t force_slab, int ktile)
{
    BuildLayout L{};
    L.nao = p.nao;
    L.naux_pad = p.naux_pad;
    L.nf = p.nf_pad;
    L.ncol = with_D ? p.nao : nocc;
    L.precision = precision;
    L.with_D = with_D;
    L.crows = c_split_rows(p.nf_pad, force_slab > 0);
    L.nsplit_c = (int)((p.nf_pad + L.crows - 1) / L.crows);
    const bool fixed = force_slab > 0;
    KShape tuned{0, 0};
    if (nsplit == 0 && !with_D && !delta) {
        const auto it = p.tuned.find((int64_t)nocc * 8 + precision);
        if (it != p.tuned.end()) tuned = it->second;
    }
    L.delta = delta;
    // aux slab of the K build: X = nao x slab x ncol elements per operand
    // bytes of X per element (both BF16 planes; int8 slices plus block scales)
    const double esz = precision == DFJK_FP64 ? 8.0
                     : precision == DFJK_MIXED_FP32 ? 4.0
                     : precision == DFJK_MIXED_BF16X3 ? 4.0 : i8_slices(precision) + 8.0 / kI8Block;
    // automatic: the largest multiple of 128 whose slab-sized buffers (X, its low part,
    // the expanded B of the density route, the second operand of the increment) stay
    // within kAutoSlabBytes
    // Overlapped slabs (C route): when the K build needs several aux slabs, the
    // half transform of slab s + 1 runs on a second stream while the K GEMM of
    // slab s runs, into the other of two X buffers (the automatic slab is
    // sized for both).  A molecule that fits one slab is not cut in two: at
    // 2,816 aux that saved 1.5% of an FP64 build, lost 3% in FP32, and the
    // GEMM shares the chip with the half transform while they overlap.  The
    // int8 GEMM, bound by operand traffic through L2, runs slabs in turn:
    // beside the half transform the 128-water build took 1.33 s, against
    // 1.21 s for the same build with sequential slabs.
    const bool may_overlap = allow_overlap && !with_D && !delta && !p.host_B && p.naux_pad >= 2 * kPadAux &&
                             !is_int8(precision);
    const double per_aux = (double)p.nao * L.ncol *
                           (esz + (with_D ? 8 : 0)) *
                           (delta ? 2 : 1) * (may_overlap ? 2 : 1);
    int64_t slab = p.host_B ? p.host_slab
                 : force_slab > 0 ? force_slab
                 : p.aux_slab > 0 ? (int64_t)align_up((size_t)p.aux_slab, kPadAux)
                                  : (int64_t)(kAutoSlabBytes / per_aux) / kPadAux * kPadAux;
    if (is_int8(precision) && !p.host_B) {   // 128 rows of int8 slices below 4 GiB (32-bit offsets)
        const int64_t ncol_e = L.ncol + (L.ncol & 1);
        const int64_t cap = ((int64_t)UINT32_MAX / (128 * kI8Slices) / ncol_e) / kPadAux * kPadAux;
        if (slab > cap) slab = cap;
        // an int8 build that needs several automatic slabs takes slabs of at
        // most 1,024 aux: on the 128-water cluster (640 orbitals) 512 / 768 /
        // 1024 / 1536 / 2048 / 3840 aux per slab measured 1.17 / 1.16 / 1.15 /
        // 1.18 / 1.28 / 1.43 s per build (the GEMM's k range per workgroup
        // grows with the slab).  A molecule that fits one slab keeps it.
        if (force_slab <= 0 && p.aux_slab <= 0 && slab < p.naux_pad && slab > kI8AutoSlab) slab = kI8AutoSlab;
    }
    if (slab < kPadAux) slab = kPadAux;
    if (slab > p.naux_pad) slab = p.naux_pad;
    L.slab = slab;
    L.nslab = (p.naux_pad + slab - 1) / slab;
    L.overlap = may_overlap && L.nslab >= 2;
    L.j_side = allow_overlap && !p.host_B;
    L.kdim = x_kdim(precision, slab, L.ncol);
    // Tile width of the K contraction: for FP64 (C and density routes) and FP32
    // the rule of syrk_tile_width, for int8_fast that of i8_fast_tile; for FP64
    // the autotuner's choice for the shape, or the caller's, wins.  int8, BF16x3
    // and every increment keep 128.
    // With a forced slab (the static scratch) the built-in shapes are those of the
    // smallest partial tiles: 64-wide FP64 tiles where 128-wide ones execute over 14%
    // more products, else 128, and no more splits than one per 256 k.
    L.ktile = kTileK;
    if (fixed && precision == DFJK_FP64) {
        auto executed = [&](int64_t t) { const int64_t n = (p.nao + t - 1) / t; return n * (n + 1) / 2 * t * t; };
        const int kt = p.k_tile != 0 ? p.k_tile : tuned.tile;
        if (kt == 64 || kt == 96) L.ktile = kt;
        else if (kt == 0 && (double)executed(kTileK) > 1.14 * (double)executed(64)) L.ktile = 64;
    } else if ((precision == DFJK_FP64 || precision == DFJK_MIXED_FP32) && !delta && !fixed) {
        int kt = ktile;
        if (kt == 0 && precision == DFJK_FP64) kt = p.k_tile;
        if (kt == 0) kt = tuned.tile;
        L.ktile = kt == 64 || kt == 96 || kt == kTileK ? kt : syrk_tile_width(p.nao, L.kdim, precision == DFJK_FP64, p.num_cus);
    }
    if (fixed && (precision == DFJK_MIXED_FP32 || precision == DFJK_MIXED_INT8_FAST) && tuned.tile != 0)
        L.ktile = tuned.tile;
    if (precision == DFJK_MIXED_INT8_FAST && !delta && !fixed) {
        const int kt = ktile != 0 ? ktile : tuned.tile;
        L.ktile = kt == 64 || kt == kTileK ? kt : i8_fast_tile(p.nao);
    }
    L.ntile = (int)((p.nao + L.ktile - 1) / L.ktile);
    const int ntiles = delta ? L.ntile * L.ntile : L.ntile * (L.ntile + 1) / 2;
    // FP64 and FP32 syrk: enough splits for 32 workgroups per CU with 96-wide tiles, 64
    // with 64-wide ones (32 in FP64 up to 640 AO, where more lengthen the reduction by as much)
    // and 16 with 128-wide ones.  Whole builds, ms: 64-wide 600 AO 144 / 288 splits 1.90 /
    // 1.93, 840 AO 72 / 144 6.62 / 6.35, 960 AO 64 / 128 9.24 / 9.13, 1,080 AO 48 / 96 16.05 /
    // 15.84; 96-wide 960 AO 72 / 144 / 288 9.13 / 8.92 / 9.08; K alone: 1,920 AO on 96-wide,
    // 16 / 32 / 72 89.9 / 85.4 / 84.1; 3,840 AO on 128-wide, 4 / 8 / 16 179 / 168 / 168.  A
    // split count of 8 or more is rounded down to a multiple of the XCD count,
    // so that the syrk runs whole splits per XCD.  In FP32 they are parts of the
    // mixed_nsplit ranges in which the FP32 sums fold; the increment, whose reduction
    // costs more per split, keeps whole ranges (360 / 480 / 600 AO with parts 2.28 / 3.73 /
    // 5.48 ms, without 1.63 / 2.46 / 4.10), and a build in many slabs, whose k ranges are
    // short already, takes fewer parts (1,920 AO in 44 slabs: 28 splits a slab 19.4 GB and
    // 78.8 ms, 8 splits 5.5 GB and 75.3).
    const int many = xcd_round(choose_ksplit(ntiles, L.kdim, p.num_cus,
                                             L.ktile == kTileK ? 16
                                             : precision == DFJK_FP64 && !fixed && (L.ktile == 96 || p.nao <= 640) ? 32
                                                                                                                   : 64,
                                             !fixed, delta));
    L.nsub = 1;
    if (precision == DFJK_FP64) {
        L.nsplit_k = many;
    } else if (is_int8(precision)) {
        L.nsplit_k = i8_nsplit(p.nao, L.kdim, !delta, L.ktile, p.num_cus);
    } else {
        L.nsplit_k = mixed_nsplit(p.nao, L.kdim, !delta, p.num_cus);
        if (precision == DFJK_MIXED_FP32 && !fixed && !delta) {
            const double whole = (double)L.nslab * L.nsplit_k * ntiles * L.ktile * L.ktile * 8;   // bytes without parts
            const int64_t fit = (int64_t)std::min(1e6, kPartBytes / whole);
            L.nsub = f32_parts(L.kdim, L.nsplit_k, std::min<int64_t>((many + L.nsplit_k / 2) / L.nsplit_k, fit));
            L.nsplit_k *= L.nsub;
        }
    }
    if (nsplit == 0) nsplit = tuned.nsplit;   // a split count the autotuner measured for this shape
    if (nsplit > 0) {   // a batch (or the autotuner) chooses the split count
        if (precision == DFJK_MIXED_FP32 && !fixed && !delta) {   // parts of the same ranges: no fold moves
            const int ranges = L.nsplit_k / L.nsub;
            L.nsub = f32_parts(L.kdim, ranges, nsplit / ranges);
            L.nsplit_k = ranges * L.nsub;
        } else {
            L.nsplit_k = (int)std::min<int64_t>(nsplit, std::max<int64_t>(L.kdim / 256, L.nsplit_k));
        }
    }
    size_t off = 0;
    auto take = [&](size_t bytes) {
        off = align_up(off, 256);
        const size_t o = off;
        off += bytes;
        return o;
    };
    L.o_D = take((size_t)p.nao * p.nao * 8);
    L.o_cpart = take((size_t)L.nsplit_c * p.naux_pad * 8);
    L.o_c = take((size_t)p.naux_pad * 8);
    const size_t nx = (size_t)p.nao * L.kdim;
    const size_t xb = x_bytes(precision, p.nao, L.kdim), xlo = x_lo_bytes(precision, p.nao, L.kdim);
    L.o_X = take(xb);
    L.o_Xlo = xlo ? take(xlo) : 0;
    L.o_Bfull = with_D ? take(nx * 8) : 0;
    const size_t cpad = (size_t)(p.nao + 1) * ht_ldc(L.ncol) * 8;
    L.o_Cp = take(cpad);
    L.o_Cp2 = delta ? take(cpad) : 0;
    if (L.overlap) {
        L.o_Xb = take(xb);
        L.o_Xblo = xlo ? take(xlo) : 0;
    }
    if (delta) {
        L.o_X2 = take(xb);
        L.o_X2lo = xlo ? take(xlo) : 0;
        L.o_U = take((size_t)p.nao * nocc * 8);
        L.o_W = take((size_t)p.nao * nocc * 8);
        L.o_Cr = take((size_t)p.nao * nocc * 8);
        L.o_align = take(align_work_doubles(nocc) * 8);
    }
    L.o_Kpart = take((size_t)L.nslab * L.nsplit_k * ntiles * L.ktile * L.ktile * 8);
    if (p.host_B) {   // two staging buffers for slabs of the host-resident B
        L.o_stage[0] = take((size_t)p.nf_pad * L.slab * 8);
        L.o_stage[1] = take((size_t)p.nf_pad * L.slab * 8);
    }
    L.o_Epart = take((size_t)L.ntile * (L.ntile + 1) / 2 * reduce_chunks(L.ktile) * 8);
    L.bytes = align_up(off, 256);
    return L;
}

bool static_layout(const Plan &p, int32_t nocc, int32_t precision, bool with_D, BuildLayout &L)
{
    for (const int nsplit : {0, -1}) {   // the tuned shape, then the built-in one
        for (int64_t slab = p.naux_pad; slab >= kPadAux; slab -= kPadAux) {
            L = build_layout(p, nocc, precision, with_D, false, nsplit, false, slab);
            if (L.bytes <= DFJK_STATIC_SCRATCH_BYTES) return true;
            if (p.host_B) break;   // the slab of a host-resident B is fixed
        }
    }
    return false;
}

// Autotuner candidates.  Split counts are half, one, two and four times the built-in
// choice of each tile, below 28,000 (the ABI's code is 1000 * tile + splits, and the
// tiles 96 and 128 are that far apart); the FP64 and FP32 syrk also try 64- and 96-wide tiles and int8_fast 64-wide ones, which leave
// less of the work above the diagonal or past nao.  Each is the shape that its own
// layout has.
std::vector<KShape> autotune_candidates(const Plan &p, int32_t nocc, int32_t precision)
{
    std::vector<KShape> c;
    std::vector<int> tiles = {kTileK};
    if (precision == DFJK_FP64 || precision == DFJK_MIXED_FP32) { tiles.push_back(64); tiles.push_back(96); }
    if (precision == DFJK_MIXED_INT8_FAST) tiles.push_back(64);
    for (int kt : tiles) {
        const int built_in = build_layout(p, nocc, precision, false, false, -1, true, 0, kt).nsplit_k;
        for (int f : {-2, 1, 2, 4}) {
            int n = std::min(std::max(f < 0 ? built_in / 2 : built_in * f, 1), 27999);
            if (precision == DFJK_FP64 && n >= kXcds) n = n / kXcds * kXcds;   // whole splits per XCD
            n = build_layout(p, nocc, precision, false, false, n, true, 0, kt).nsplit_k;
            if (std::none_of(c.begin(), c.end(), [&](const KShape &k) { return k.tile == kt && k.nsplit == n; }))
                c.push_back({kt, n});
        }
    }
    return c;
}

void launch_gemm_bf16x3(bool lower, const void *A, const void *Alo, const void *B, const void *Blo, int64_t nao,
                        int64_t kdim, int nsplit, double *part, hipStream_t s);

// c for plen aux functions of B (rows ld = plen apart) from the density, and J
// zeroed first where jzero is given.
static void launch_c(const Plan &p, const BuildLayout &L, const double *B, int64_t plen, const double *D, double *c,
                     double *jzero, char *scratch, hipStream_t s)
{
    double *cpart = reinterpret_cast<double *>(scratch + L.o_cpart);
    const int64_t njj = jzero ? p.nao * p.nao : 0;
    hipLaunchKernelGGL(k_c_partial, dim3((unsigned)((plen + kCCols - 1) / kCCols), L.nsplit_c), dim3(256), 0, s, B,
                       plen, D, p.nao, p.d.f_mu, p.d.f_nu, p.d.f_w, p.nf, p.nf_pad, L.crows, cpart);
    hipLaunchKernelGGL(k_c_sum, dim3(c_sum_blocks(plen, njj)), dim3(1024), 0, s, cpart, (int64_t)L.nsplit_c, plen, c,
                       jzero, njj);
}

static void launch_j_rows(const Plan &p, const double *B, int64_t ld, const double *c, bool accumulate, double *J,
                          hipStream_t s)
{
    if (p.nf > 0)
        hipLaunchKernelGGL(k_j_rows, dim3((unsigned)((p.nf + 3) / 4)), dim3(256), 0, s, B, ld, c, p.d.f_mu, p.d.f_nu,
                           p.d.f_w, p.nf, p.nao, accumulate ? 1 : 0, J);
}

// J from the resident B and the density (steps 2-3).
static void launch_j(Plan &p, const BuildLayout &L, const double *D, double *J, char *scratch, hipStream_t s)
{
    double *cvec = reinterpret_cast<double *>(scratch + L.o_c);
    p.prof.stream = s;
    p.prof.mark(ST_J, true);
    launch_c(p, L, p.d.B, p.naux_pad, D, cvec, J, scratch, s);
    launch_j_rows(p, p.d.B, p.naux_pad, cvec, false, J, s);
    p.prof.mark(ST_J, false);
}

// Arguments of the steps around the half transform for one molecule with ncol
// coefficient columns (dmode, scale: the density in D, see PreArgs).
static PreArgs pre_args(const Plan &p, const BuildLayout &L, const double *C, int64_t ncol, int dmode, double scale,
                        double *D, double *J, char *scratch)
{
    PreArgs a{};
    a.C = C; a.D = D; a.J = J;
    a.Cp = reinterpret_cast<double *>(scratch + L.o_Cp);
    a.f_mu = p.d.f_mu; a.f_nu = p.d.f_nu; a.f_w = p.d.f_w; a.B = p.d.B;
    a.cpart = reinterpret_cast<double *>(scratch + L.o_cpart);
    a.cvec = reinterpret_cast<double *>(scratch + L.o_c);
    a.scale = scale;
    a.nao = p.nao; a.nf = p.nf; a.nf_pad = p.nf_pad; a.ld = p.naux_pad;
    a.ncol = (int32_t)ncol; a.ldc = (int32_t)ht_ldc(ncol); a.dmode = dmode;
    a.crows = L.crows; a.nsplit_c = L.nsplit_c;
    return a;
}

static void launch_prep(const PreArgs &a, hipStream_t s)
{
    hipLaunchKernelGGL(k_prep, dim3(prep_blocks(a)), dim3(256), 0, s, a, density_blocks(a));
}

// The zero-padded copy of the coefficients that the half transform reads
// (k_pad_coef), in the build scratch at `off`.
static const double *pad_coef(const Plan &p, const double *C, int32_t ncol, char *scratch, size_t off, hipStream_t s)
{
    double *Cp = reinterpret_cast<double *>(scratch + off);
    const int64_t ldc = ht_ldc(ncol), n = (p.nao + 1) * ldc;
    hipLaunchKernelGGL(k_pad_coef, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, C, p.nao, ncol, (int32_t)ldc,
                       Cp);
    return Cp;
}

// Half transform of one aux slab of B (rows ld apart) with padded coefficients Cp.
static HTArgs ht_args(const Plan &p, int precision, const double *B, int64_t ld, const double *Cp, int32_t ncol,
                      int64_t p_begin, int64_t plen, void *X, void *Xlo)
{
    return HTArgs{B, ld, Cp, ncol, (int32_t)ht_ldc(ncol), p.d.hk_off, p.d.hk_row, p.d.hk_nu, X, Xlo, p_begin, plen,
                  p.d.hk_order, i8_slices(precision)};
}

static void launch_ht(const Plan &p, int precision, const double *B, int64_t ld, const double *Cp, int32_t ncol,
                      int64_t p_begin, int64_t plen, void *X, void *Xlo, hipStream_t s)
{
    dispatch_halftrans(precision, ht_args(p, precision, B, ld, Cp, ncol, p_begin, plen, X, Xlo), p.nao, s);
}

// Steps 5-6 for every aux slab: the half transform of C1 (and of C2 for the
// increment, which contracts X(C1) with X(C2) over all tiles), then the slab's
// K contribution into its own split-K partials: lower tiles of X X^T (C route),
// X B~^T (density route, B~ the expanded tensor) or every tile of X1 X2^T.
// ncol <= L.ncol columns; slabs reuse the X buffers and the stream orders them.
static void slab_gemm(const BuildLayout &L, bool lower, const void *X, const void *Xlo, const void *Bop,
                      const void *Bop_lo, int64_t nao, int64_t kdim, double *part, hipStream_t s)
{
    if (L.precision == DFJK_FP64) {
        const int64_t ksplit = (int64_t)align_up((size_t)((kdim + L.nsplit_k - 1) / L.nsplit_k), 16);
        launch_syrk_f64(lower, static_cast<const double *>(X), static_cast<const double *>(Bop), nao, kdim, ksplit,
                        L.nsplit_k, L.ktile, part, s);
    } else if (L.precision == DFJK_MIXED_FP32) {
        const int ranges = L.nsplit_k / L.nsub;
        const int64_t ksplit = (int64_t)align_up((size_t)((kdim + ranges - 1) / ranges), 32);
        launch_syrk_f32(lower, static_cast<const float *>(X), static_cast<const float *>(Bop), nao, kdim, ksplit,
                        L.nsplit_k, L.nsub, L.ktile, part, s);
    } else if (is_int8(L.precision)) {
        launch_gemm_i8(lower, X, static_cast<const double *>(Xlo), Bop, static_cast<const double *>(Bop_lo), nao,
                       kdim, L.nsplit_k, L.precision == DFJK_MIXED_INT8_FAST, L.ktile, part, s);
    } else {
        launch_gemm_bf16x3(lower, X, Xlo, Bop, Bop_lo, nao, kdim, L.nsplit_k, part, s);
    }
}

// The overlapped schedule of a C-route contraction: the half transform of
// slab s goes to the plan's second stream into X buffer s % 2, after the K
// GEMM that last read that buffer; the GEMM of slab s waits for it on `s`.
// Every side-stream launch is joined back into `s` by the GEMM's wait.
static bool overlap_streams(Plan &p)
{
    if (p.ht_stream) return true;
    hipEvent_t ev[5] = {};
    hipStream_t hs = nullptr;
    bool ok = true;
    for (hipEvent_t &e : ev) ok = ok && hipEventCreateWithFlags(&e, hipEventDisableTiming) == hipSuccess;
    ok = ok && hipStreamCreateWithFlags(&hs, hipStreamNonBlocking) == hipSuccess;
    if (!ok) {   // fall back to the single-stream schedule
        for (hipEvent_t e : ev)
            if (e) (void)hipEventDestroy(e);
        if (hs) (void)hipStreamDestroy(hs);
        return false;
    }
    p.ev_fork = ev[0]; p.ev_ht[0] = ev[1]; p.ev_ht[1] = ev[2]; p.ev_kdone[0] = ev[3]; p.ev_kdone[1] = ev[4];
    p.ht_stream = hs;
    return true;
}

static void contract_slabs_overlapped(Plan &p, const BuildLayout &L, int64_t ncol, char *scratch, hipStream_t s)
{
    const int64_t nao = p.nao, ld = p.naux_pad;
    Profiler &pr = p.prof;
    void *X[2] = {scratch + L.o_X, scratch + L.o_Xb};
    void *Xlo[2] = {L.o_Xlo ? scratch + L.o_Xlo : nullptr, L.o_Xblo ? scratch + L.o_Xblo : nullptr};
    double *Kpart = reinterpret_cast<double *>(scratch + L.o_Kpart);
    const int ntiles = L.ntile * (L.ntile + 1) / 2;
    const size_t slab_part = (size_t)L.nsplit_k * ntiles * L.ktile * L.ktile;
    hipStream_t hs = p.ht_stream;
    const double *Cp = reinterpret_cast<const double *>(scratch + L.o_Cp);
    (void)hipEventRecord(p.ev_fork, s);
    (void)hipStreamWaitEvent(hs, p.ev_fork, 0);
    auto ht = [&](int64_t sl) {
        const int b = (int)(sl & 1);
        const int64_t pb = sl * L.slab, plen = (ld - pb < L.slab) ? ld - pb : L.slab;
        if (sl >= 2) (void)hipStreamWaitEvent(hs, p.ev_kdone[b], 0);
        pr.stream = hs;
        pr.mark(ST_HALFTRANS, true);
        launch_ht(p, L.precision, p.d.B, ld, Cp, (int32_t)ncol, pb, plen, X[b], Xlo[b], hs);
        pr.mark(ST_HALFTRANS, false);
        pr.stream = s;
        (void)hipEventRecord(p.ev_ht[b], hs);
    };
    ht(0);
    for (int64_t sl = 0; sl < L.nslab; ++sl) {
        const int b = (int)(sl & 1);
        const int64_t pb = sl * L.slab, plen = (ld - pb < L.slab) ? ld - pb : L.slab;
        if (sl + 1 < L.nslab) ht(sl + 1);
        (void)hipStreamWaitEvent(s, p.ev_ht[b], 0);
        pr.mark(ST_K, true);
        slab_gemm(L, true, X[b], Xlo[b], X[b], Xlo[b], nao, x_kdim(L.precision, plen, ncol), Kpart + sl * slab_part,
                  s);
        pr.mark(ST_K, false);
        (void)hipEventRecord(p.ev_kdone[b], s);
    }
}

// The coefficients are in the scratch, zero-padded (k_prep; the increment's two
// here).
static void contract_slabs(Plan &p, const BuildLayout &L, const double *C1, const double *C2, int64_t ncol,
                           char *scratch, hipStream_t s)
{
    if (L.overlap && C2 == nullptr && overlap_streams(p)) {
        contract_slabs_overlapped(p, L, ncol, scratch, s);
        return;
    }
    const int64_t nao = p.nao, ld = p.naux_pad;
    Profiler &pr = p.prof;
    void *X = scratch + L.o_X;
    void *Xlo = L.o_Xlo ? scratch + L.o_Xlo : nullptr;
    double *Bt = L.o_Bfull ? reinterpret_cast<double *>(scratch + L.o_Bfull) : nullptr;
    double *Kpart = reinterpret_cast<double *>(scratch + L.o_Kpart);
    const bool lower = !L.delta;
    const int ntiles = lower ? L.ntile * (L.ntile + 1) / 2 : L.ntile * L.ntile;
    const size_t slab_part = (size_t)L.nsplit_k * ntiles * L.ktile * L.ktile;
    void *X2 = L.delta ? scratch + L.o_X2 : nullptr;
    void *X2lo = L.o_X2lo ? scratch + L.o_X2lo : nullptr;
    const double *Cp1 = L.delta ? pad_coef(p, C1, (int32_t)ncol, scratch, L.o_Cp, s)
                                : reinterpret_cast<const double *>(scratch + L.o_Cp);
    const double *Cp2 = L.delta ? pad_coef(p, C2, (int32_t)ncol, scratch, L.o_Cp2, s) : nullptr;
    for (int64_t sl = 0; sl < L.nslab; ++sl) {
        const int64_t pb = sl * L.slab, plen = (ld - pb < L.slab) ? ld - pb : L.slab;
        const int64_t kdim = x_kdim(L.precision, plen, ncol);
        pr.mark(ST_HALFTRANS, true);
        launch_ht(p, L.precision, p.d.B, ld, Cp1, (int32_t)ncol, pb, plen, X, Xlo, s);
        if (L.norms)
            launch_i8_norms(X, static_cast<const double *>(Xlo), nao, kdim, reinterpret_cast<double *>(scratch + L.o_norms),
                            s);
        if (L.delta)
            launch_ht(p, L.precision, p.d.B, ld, Cp2, (int32_t)ncol, pb, plen, X2, X2lo, s);
        else if (L.with_D)
            hipLaunchKernelGGL(k_expand_B, dim3((unsigned)(plen / kExpP), (unsigned)nao), dim3(256), 0, s,
                               p.d.B, ld, p.d.hk_off, p.d.hk_row, p.d.hk_nu, nao, pb, plen, Bt);
        pr.mark(ST_HALFTRANS, false);
        pr.mark(ST_K, true);
        const void *Bop = L.delta ? (const void *)X2 : (L.with_D ? (const void *)Bt : (const void *)X);
        const void *Bop_lo = L.delta ? (const void *)X2lo : Xlo;
        slab_gemm(L, lower, X, Xlo, Bop, Bop_lo, nao, kdim, Kpart + sl * slab_part, s);
        pr.mark(ST_K, false);
    }
}

// The plan's side stream and its fork / join events (created on first use;
// false if HIP refuses, and the caller then runs the work in turn on its
// own stream).  A build runs J there; a setup runs the integrals there.
bool side_stream(Plan &p)
{
    if (p.j_stream) return true;
    hipEvent_t a = nullptr, b = nullptr;
    hipStream_t js = nullptr;
    bool ok = hipEventCreateWithFlags(&a, hipEventDisableTiming) == hipSuccess &&
              hipEventCreateWithFlags(&b, hipEventDisableTiming) == hipSuccess &&
              hipStreamCreateWithFlags(&js, hipStreamNonBlocking) == hipSuccess;
    if (!ok) {
        if (a) (void)hipEventDestroy(a);
        if (b) (void)hipEventDestroy(b);
        if (js) (void)hipStreamDestroy(js);
        return false;
    }
    p.ev_jfork = a; p.ev_jdone = b; p.j_stream = js;
    return true;
}

// J of one call on the plan's side stream, from side_begin to side_end (the lock is
// held between them), joined into the caller's stream by side_join.  js is the
// caller's stream where the side stream is not wanted or not to be had.
struct SideJ {
    hipStream_t js;
    bool on = false;
    std::pair<hipEvent_t, hipEvent_t> ev{};
    std::unique_lock<std::mutex> lock;
};

// Whether a stream capture that s is not part of holds the side stream.
static bool captured_elsewhere(hipStream_t js, hipStream_t s)
{
    hipStreamCaptureStatus cj = hipStreamCaptureStatusNone, cs = hipStreamCaptureStatusNone;
    unsigned long long ij = 0, is = 0;
    if (hipStreamGetCaptureInfo(js, &cj, &ij) != hipSuccess) return true;
    if (cj == hipStreamCaptureStatusNone) return false;
    if (s == nullptr || hipStreamGetCaptureInfo(s, &cs, &is) != hipSuccess) return true;
    return cs != hipStreamCaptureStatusActive || ij != is;
}

// js waits for what s holds by now.
static void side_wait(const SideJ &j, hipStream_t s)
{
    (void)hipEventRecord(j.ev.first, s);
    (void)hipStreamWaitEvent(j.js, j.ev.first, 0);
}

static SideJ side_begin(Plan &p, hipStream_t s, bool want)
{
    SideJ j;
    j.js = s;
    if (!want) return j;
    std::unique_lock<std::mutex> lock(p.side_mu);
    if (!side_stream(p) || captured_elsewhere(p.j_stream, s)) return j;
    if (!p.side_events.empty()) {
        j.ev = p.side_events.back();
        p.side_events.pop_back();
    } else {
        if (hipEventCreateWithFlags(&j.ev.first, hipEventDisableTiming) != hipSuccess) return j;
        if (hipEventCreateWithFlags(&j.ev.second, hipEventDisableTiming) != hipSuccess) {
            (void)hipEventDestroy(j.ev.first);
            return j;
        }
    }
    j.on = true;
    j.js = p.j_stream;
    j.lock = std::move(lock);
    side_wait(j, s);
    return j;
}

static void side_end(SideJ &j)
{
    if (!j.on) return;
    (void)hipEventRecord(j.ev.second, j.js);
    j.lock.unlock();
}

static void side_join(Plan &p, SideJ &j, hipStream_t s)
{
    if (!j.on) return;
    (void)hipStreamWaitEvent(s, j.ev.second, 0);
    std::lock_guard<std::mutex> lock(p.side_mu);
    p.side_events.push_back(j.ev);
}

void launch_build(Plan &p, const BuildLayout &L, const double *C, const double *Din, double *J, double *K,
                  double *E, char *scratch, hipStream_t s)
{
    const int64_t nao = p.nao, ld = p.naux_pad;
    double *D = reinterpret_cast<double *>(scratch + L.o_D);
    double *cvec = reinterpret_cast<double *>(scratch + L.o_c);
    double *Kpart = reinterpret_cast<double *>(scratch + L.o_Kpart);
    double *Epart = reinterpret_cast<double *>(scratch + L.o_Epart);
    Profiler &pr = p.prof;
    pr.stream = s;
    pr.mark(ST_BUILD, true);

    // J streams B through HBM twice while the half transform and K are bound by the
    // matrix pipes: with a B of kJSideBytes or more the density and J run on a side
    // stream from the start, joined before the energies.  Beside the half
    // transform, J costs 32 waters 0.3 ms (2.15 -> 2.47 ms); beside K it cost 0.7 (6.6 ->
    // 7.35 ms), more than the 0.5 that it takes alone.  J reads D and B and writes
    // only J and its own scratch.
    SideJ side = side_begin(p, s, L.j_side && (double)p.nf_pad * p.naux_pad * 8.0 >= kJSideBytes);
    const bool jside = side.on;
    hipStream_t js = side.js;
    pr.mark(ST_DENSITY, true);
    const int dmode = L.with_D ? 2 : L.delta || jside ? 0 : 1;   // the density where k_prep does not form it
    if (!L.with_D && dmode == 0) launch_density(C, nao, (int32_t)L.ncol, 2.0, D, js);
    const double *C1 = nullptr, *C2 = nullptr;
    if (L.delta) {   // U, W from C rotated onto C0 (D is unchanged by the rotation)
        double *Cr = reinterpret_cast<double *>(scratch + L.o_Cr);
        double *U = reinterpret_cast<double *>(scratch + L.o_U), *W = reinterpret_cast<double *>(scratch + L.o_W);
        launch_align(C, L.C0, nao, (int32_t)L.ncol, reinterpret_cast<double *>(scratch + L.o_align), Cr, s);
        hipLaunchKernelGGL(k_uw, dim3((unsigned)((nao * L.ncol + 255) / 256)), dim3(256), 0, s, Cr, L.C0, nao,
                           (int32_t)L.ncol, U, W);
        C1 = U;
        C2 = W;
    } else {
        launch_prep(pre_args(p, L, L.with_D ? Din : C, L.ncol, dmode, 2.0, D, J, scratch), s);
        if (jside && L.with_D) side_wait(side, s);   // D is copied by then
    }
    pr.mark(ST_DENSITY, false);
    launch_j(p, L, D, J, scratch, js);
    pr.stream = s;
    side_end(side);
    contract_slabs(p, L, C1, C2, L.ncol, scratch, s);
    side_join(p, side, s);
    // split-K sum, mirror, energies (after the side stream: they read D and c)
    pr.mark(ST_KREDUCE, true);
    const int nlower = L.ntile * (L.ntile + 1) / 2;
    const int64_t nep = (int64_t)nlower * (L.delta ? kTileK / 16 : reduce_chunks(L.ktile));   // energy partials
    if (L.delta)
        hipLaunchKernelGGL(k_k_reduce_delta, dim3(nlower, kTileK / 16), dim3(256), 0, s, Kpart,
                           (int)(L.nslab * L.nsplit_k),
                           L.ntile, nao, L.K0, D, K, Epart);
    else
        hipLaunchKernelGGL(k_k_reduce, dim3(nlower, reduce_chunks(L.ktile)), dim3(256), 0, s, Kpart,
                           (int)(L.nslab * L.nsplit_k), L.ntile, L.ktile, nao, L.with_D ? 1.0 : 2.0, D, K, Epart);
    hipLaunchKernelGGL(k_energies, dim3(1), dim3(256), 0, s, cvec, ld, Epart, nep, -0.25, E);
    pr.mark(ST_KREDUCE, false);
    pr.mark(ST_BUILD, false);
}

BuildLayout build_layout_uks(const Plan &p, int32_t nocc_a, int32_t nocc_b, int32_t precision)
{
    BuildLayout L = build_layout(p, nocc_a > nocc_b ? nocc_a : nocc_b, precision, false);
    L.uks = true;
    L.nocc_a = nocc_a;
    L.nocc_b = nocc_b;
    size_t off = L.bytes;
    auto take = [&](size_t bytes) {
        off = align_up(off, 256);
        const size_t o = off;
        off += bytes;
        return o;
    };
    L.o_Da = take((size_t)p.nao * p.nao * 8);
    L.o_Db = take((size_t)p.nao * p.nao * 8);
    L.o_Epart = take((size_t)2 * L.ntile * (L.ntile + 1) / 2 * reduce_chunks(L.ktile) * 8);   // one block per spin
    L.bytes = align_up(off, 256);
    return L;
}

// Open-shell build: D_s = C_s C_s^T for s = alpha, beta; J from D = D_a + D_b;
// K_s = sum_P B_P D_s B_P = X_s X_s^T; E_J = 1/2 Tr D J = 1/2 sum_P c_P^2,
// E_K = -1/2 (Tr D_a K_a + Tr D_b K_b).
void launch_build_uks(Plan &p, const BuildLayout &L, const double *Ca, const double *Cb, double *J, double *Ka,
                      double *Kb, double *E, char *scratch, hipStream_t s)
{
    const int64_t nao = p.nao, ld = p.naux_pad;
    double *D = reinterpret_cast<double *>(scratch + L.o_D);
    double *Ds[2] = {reinterpret_cast<double *>(scratch + L.o_Da), reinterpret_cast<double *>(scratch + L.o_Db)};
    const double *Cs[2] = {Ca, Cb};
    double *Ks[2] = {Ka, Kb};
    const int32_t nocc[2] = {L.nocc_a, L.nocc_b};
    double *cvec = reinterpret_cast<double *>(scratch + L.o_c);
    double *Kpart = reinterpret_cast<double *>(scratch + L.o_Kpart);
    double *Epart = reinterpret_cast<double *>(scratch + L.o_Epart);
    const int nlower = L.ntile * (L.ntile + 1) / 2;
    const int64_t nep = (int64_t)nlower * reduce_chunks(L.ktile);
    Profiler &pr = p.prof;
    pr.stream = s;

    pr.mark(ST_DENSITY, true);
    for (int sp = 0; sp < 2; ++sp) {
        if (nocc[sp] > 0) launch_density(Cs[sp], nao, nocc[sp], 1.0, Ds[sp], s);
        else fill(Ds[sp], nao * nao, 0.0, s);
    }
    hipLaunchKernelGGL(k_add, dim3((unsigned)((nao * nao + 255) / 256)), dim3(256), 0, s, Ds[0], Ds[1], nao * nao, D);
    pr.mark(ST_DENSITY, false);
    // J on the side stream where B is large (as in launch_build)
    SideJ side = side_begin(p, s, L.j_side && (double)p.nf_pad * ld * 8.0 >= kJSideBytes);
    launch_j(p, L, D, J, scratch, side.js);
    pr.stream = s;
    side_end(side);
    for (int sp = 0; sp < 2; ++sp) {
        if (nocc[sp] == 0) {
            fill(Ks[sp], nao * nao, 0.0, s);
            fill(Epart + sp * nep, nep, 0.0, s);
            continue;
        }
        launch_prep(pre_args(p, L, Cs[sp], nocc[sp], 0, 1.0, Ds[sp], J, scratch), s);
        contract_slabs(p, L, nullptr, nullptr, nocc[sp], scratch, s);
        pr.mark(ST_KREDUCE, true);
        hipLaunchKernelGGL(k_k_reduce, dim3(nlower, reduce_chunks(L.ktile)), dim3(256), 0, s, Kpart,
                           (int)(L.nslab * L.nsplit_k), L.ntile, L.ktile, nao, 1.0, Ds[sp], Ks[sp], Epart + sp * nep);
        pr.mark(ST_KREDUCE, false);
    }
    side_join(p, side, s);
    pr.mark(ST_KREDUCE, true);
    hipLaunchKernelGGL(k_energies, dim3(1), dim3(256), 0, s, cvec, ld, Epart, 2 * nep, -0.5, E);
    pr.mark(ST_KREDUCE, false);
}

// FP64 split counts of a batch's molecules, by their own build layouts: every
// workgroup of the grouped syrk about the same k length, so that the batch has
// about 24 of them per CU (16 molecules of 1-12 waters: one count for all, for 2
// workgroups per CU of 128-wide tiles, left up to 432 chunks in a row to one
// workgroup: 1.30 ms against a floor of 0.75).
void batch_nsplits(const Plan *const *plans, int n, const BuildLayout *Ls, int *ns)
{
    double work = 0.0;
    int cus = 256;
    for (int i = 0; i < n; ++i) {
        const double nt = Ls[i].ntile * (Ls[i].ntile + 1) / 2;
        work += nt * Ls[i].ktile * Ls[i].ktile / 4096.0 * (double)Ls[i].kdim;
        cus = plans[i]->num_cus;
    }
    const double per = std::max(256.0, work / (24.0 * cus));   // k of a 64-wide tile's workgroup
    for (int i = 0; i < n; ++i) {
        const double k = std::max(256.0, per * 4096.0 / ((double)Ls[i].ktile * Ls[i].ktile));
        ns[i] = (int)std::min<int64_t>(xcd_round((int)std::max(1.0, (double)Ls[i].kdim / k + 0.5)),
                                       std::max<int64_t>(1, Ls[i].kdim / 256));
    }
}

// A batch of closed-shell builds on one stream.  The FP64, int8 and int8_fast
// molecules whose X fits one slab share launches of every step: density and padded
// coefficients, half transforms (by fragment count), c and J, K (by tile width).  The
// others (FP32, BF16x3, several slabs) form and contract X on their own, J beside them.
// Then one grouped split-K reduction and one grouped energy launch for all.
void launch_build_batch(int n, Plan *const *plans, const BuildLayout *Ls, const double *const *C, double *const *J,
                        double *const *K, double *const *E, char *const *scratch, hipStream_t s)
{
    std::vector<std::pair<Plan *, SideJ>> joins;
    std::vector<PreArgs> pre;
    std::vector<std::pair<HTArgs, int64_t>> hts, hts8;   // arguments and AO count of each grouped half transform
    std::vector<const void *> i8x;                        // grouped int8 K: slices, scales, sizes, splits, partials
    std::vector<const double *> i8s;
    std::vector<int64_t> i8m, i8k;
    std::vector<int> i8n, i8t;
    std::vector<double *> i8p;
    bool i8fast = false;
    std::vector<const double *> kx;
    std::vector<double *> kp;
    std::vector<int64_t> km, kk, ks;
    std::vector<int> ns, kt;
    for (int i = 0; i < n; ++i) {
        Plan &p = *plans[i];
        const BuildLayout &L = Ls[i];
        char *sc = scratch[i];
        const int64_t nao = p.nao;
        double *D = reinterpret_cast<double *>(sc + L.o_D);
        if (L.nslab == 1 && (L.precision == DFJK_FP64 || is_int8(L.precision))) {
            // density, padded coefficients, c and J in shared launches, the half
            // transforms and K grouped between them
            const PreArgs a = pre_args(p, L, C[i], L.ncol, 1, 2.0, D, J[i], sc);
            pre.push_back(a);
            if (is_int8(L.precision)) {
                void *Xlo = sc + L.o_Xlo;   // block scales
                hts8.emplace_back(ht_args(p, L.precision, p.d.B, p.naux_pad, a.Cp, (int32_t)L.ncol, 0, p.naux_pad,
                                          sc + L.o_X, Xlo),
                                  nao);
                i8x.push_back(sc + L.o_X);
                i8s.push_back(static_cast<const double *>(Xlo));
                i8m.push_back(nao);
                i8k.push_back(x_kdim(L.precision, p.naux_pad, L.ncol));
                i8n.push_back(L.nsplit_k);
                i8t.push_back(L.ktile);
                i8p.push_back(reinterpret_cast<double *>(sc + L.o_Kpart));
                i8fast = L.precision == DFJK_MIXED_INT8_FAST;
                continue;
            }
            hts.emplace_back(ht_args(p, DFJK_FP64, p.d.B, p.naux_pad, a.Cp, (int32_t)L.ncol, 0, p.naux_pad,
                                     sc + L.o_X, nullptr),
                             nao);
            kx.push_back(reinterpret_cast<const double *>(sc + L.o_X));
            km.push_back(nao);
            kk.push_back(L.kdim);
            ks.push_back((int64_t)align_up((size_t)((L.kdim + L.nsplit_k - 1) / L.nsplit_k), 16));
            ns.push_back(L.nsplit_k);
            kt.push_back(L.ktile);
            kp.push_back(reinterpret_cast<double *>(sc + L.o_Kpart));
            continue;
        }
        p.prof.stream = s;
        p.prof.mark(ST_DENSITY, true);
        launch_prep(pre_args(p, L, C[i], L.ncol, 1, 2.0, D, J[i], sc), s);
        p.prof.mark(ST_DENSITY, false);
        // J on the plan's side stream beside the other molecules' work,
        // joined before the energies (the only later step that reads c)
        SideJ side = side_begin(p, s, true);
        launch_j(p, L, D, J[i], sc, side.js);
        p.prof.stream = s;
        side_end(side);
        joins.emplace_back(&p, std::move(side));
        contract_slabs(p, L, nullptr, nullptr, L.ncol, sc, s);
    }
    launch_pre_group(PRE_PREP, pre, s);
    // the half transforms of the one-slab molecules, grouped by output and fragment count
    launch_halftrans_groups<OUT_F64>(hts, s);
    launch_halftrans_groups<OUT_I8>(hts8, s);
    launch_pre_group(PRE_CPART, pre, s);
    launch_pre_group(PRE_CSUM, pre, s);
    launch_pre_group(PRE_JROWS, pre, s);
    for (int T : {64, 128}) {   // one grouped int8 K per tile width
        std::vector<const void *> gx;
        std::vector<const double *> gs;
        std::vector<int64_t> gm, gk;
        std::vector<int> gn;
        std::vector<double *> gp;
        for (size_t i = 0; i < i8x.size(); ++i)
            if (i8t[i] == T) {
                gx.push_back(i8x[i]); gs.push_back(i8s[i]); gm.push_back(i8m[i]); gk.push_back(i8k[i]);
                gn.push_back(i8n[i]); gp.push_back(i8p[i]);
            }
        if (!gx.empty())
            launch_gemm_i8_group(i8fast, T, (int)gx.size(), gx.data(), gs.data(), gm.data(), gk.data(), gn.data(),
                                 gp.data(), s);
    }
    for (int T : {64, 96, 128}) {   // one grouped syrk per tile width
        std::vector<const double *> gx;
        std::vector<double *> gp;
        std::vector<int64_t> gm, gk, gs;
        std::vector<int> gn;
        for (size_t i = 0; i < kx.size(); ++i)
            if (kt[i] == T) {
                gx.push_back(kx[i]); gp.push_back(kp[i]); gm.push_back(km[i]); gk.push_back(kk[i]);
                gs.push_back(ks[i]); gn.push_back(ns[i]);
            }
        if (!gx.empty())
            launch_syrk_f64_group(T, (int)gx.size(), gx.data(), gm.data(), gk.data(), gs.data(), gn.data(),
                                  gp.data(), s);
    }
    for (int first = 0; first < n; first += kReduceGroupMax) {
        ReduceGroup grp{};
        int total = 0;
        for (int i = first; i < n && grp.n < kReduceGroupMax; ++i) {
            const BuildLayout &L = Ls[i];
            const int q = grp.n++;
            grp.blk_start[q] = total;
            grp.nsplit[q] = (int32_t)(L.nslab * L.nsplit_k);
            grp.ntm[q] = L.ntile;
            grp.T[q] = L.ktile;
            grp.nao[q] = L.nao;
            grp.part[q] = reinterpret_cast<const double *>(scratch[i] + L.o_Kpart);
            grp.D[q] = reinterpret_cast<const double *>(scratch[i] + L.o_D);
            grp.K[q] = K[i];
            grp.Epart[q] = reinterpret_cast<double *>(scratch[i] + L.o_Epart);
            total += L.ntile * (L.ntile + 1) / 2;
        }
        grp.blk_start[grp.n] = total;
        hipLaunchKernelGGL(k_k_reduce_grouped, dim3(total, reduce_chunks(kTileK)), dim3(256), 0, s, grp, 2.0);
    }
    for (auto &j : joins) side_join(*j.first, j.second, s);
    for (int first = 0; first < n; first += kEnergyGroupMax) {
        EnergyGroup grp{};
        int m = 0;
        for (int i = first; i < n && m < kEnergyGroupMax; ++i, ++m) {
            const BuildLayout &L = Ls[i];
            grp.c[m] = reinterpret_cast<const double *>(scratch[i] + L.o_c);
            grp.naux[m] = L.naux_pad;
            grp.Epart[m] = reinterpret_cast<const double *>(scratch[i] + L.o_Epart);
            grp.nEpart[m] = (int64_t)L.ntile * (L.ntile + 1) / 2 * reduce_chunks(L.ktile);
            grp.E[m] = E[i];
        }
        hipLaunchKernelGGL(k_energies_grouped, dim3(m), dim3(256), 0, s, grp, -0.25);
    }
}

// Closed-shell build from a host-resident B (paper Section 2.1: integrals in
// host memory, moved to the GPU asynchronously).  The host copy is slab-major
// ([slab][f][plen], the slab width fixed when B was offloaded); each slab is
// copied into one of two staging buffers on the plan's copy stream while the
// previous slab is consumed on `s`: c for the slab's aux functions, its
// contribution to J, the half transform and the slab's K partial tiles.
// Events order the two streams: the copy into a buffer waits for the compute
// that last read it; the compute waits for its copy.
void launch_build_hostB(Plan &p, const BuildLayout &L, const double *C, double *J, double *K, double *E,
                        char *scratch, hipStream_t s)
{
    const int64_t nao = p.nao, ld = p.naux_pad;
    double *D = reinterpret_cast<double *>(scratch + L.o_D);
    double *cvec = reinterpret_cast<double *>(scratch + L.o_c);
    double *Kpart = reinterpret_cast<double *>(scratch + L.o_Kpart);
    double *Epart = reinterpret_cast<double *>(scratch + L.o_Epart);
    double *stage[2] = {reinterpret_cast<double *>(scratch + L.o_stage[0]),
                        reinterpret_cast<double *>(scratch + L.o_stage[1])};
    void *X = scratch + L.o_X;
    void *Xlo = L.o_Xlo ? scratch + L.o_Xlo : nullptr;
    const int ntiles = L.ntile * (L.ntile + 1) / 2;
    const size_t slab_part = (size_t)L.nsplit_k * ntiles * L.ktile * L.ktile;
    Profiler &pr = p.prof;
    pr.stream = s;
    hipStream_t cs = p.copy_stream;

    auto copy_slab = [&](int64_t sl) {
        const int b = (int)(sl & 1);
        const int64_t pb = sl * L.slab, plen = (ld - pb < L.slab) ? ld - pb : L.slab;
        (void)hipStreamWaitEvent(cs, p.ev_free[b], 0);
        (void)hipMemcpyAsync(stage[b], p.hB + (size_t)p.nf_pad * pb, (size_t)p.nf_pad * plen * 8,
                             hipMemcpyHostToDevice, cs);
        (void)hipEventRecord(p.ev_ready[b], cs);
    };
    // the copy stream starts after everything already queued on s
    (void)hipEventRecord(p.ev_start, s);
    (void)hipStreamWaitEvent(cs, p.ev_start, 0);
    copy_slab(0);
    if (L.nslab > 1) copy_slab(1);

    pr.mark(ST_DENSITY, true);
    launch_prep(pre_args(p, L, C, L.ncol, 1, 2.0, D, J, scratch), s);
    pr.mark(ST_DENSITY, false);
    const double *Cp = reinterpret_cast<const double *>(scratch + L.o_Cp);
    for (int64_t sl = 0; sl < L.nslab; ++sl) {
        const int b = (int)(sl & 1);
        const int64_t pb = sl * L.slab, plen = (ld - pb < L.slab) ? ld - pb : L.slab;
        (void)hipStreamWaitEvent(s, p.ev_ready[b], 0);
        pr.mark(ST_HALFTRANS, true);
        launch_ht(p, L.precision, stage[b], plen, Cp, (int32_t)L.ncol, 0, plen, X, Xlo, s);
        if (L.norms)
            launch_i8_norms(X, static_cast<const double *>(Xlo), nao, x_kdim(L.precision, plen, L.ncol),
                            reinterpret_cast<double *>(scratch + L.o_norms), s);
        pr.mark(ST_HALFTRANS, false);
        pr.mark(ST_J, true);
        launch_c(p, L, stage[b], plen, D, cvec + pb, pb == 0 ? J : nullptr, scratch, s);
        launch_j_rows(p, stage[b], plen, cvec + pb, true, J, s);
        pr.mark(ST_J, false);
        (void)hipEventRecord(p.ev_free[b], s);      // the staging buffer is read
        if (sl + 2 < L.nslab) copy_slab(sl + 2);
        pr.mark(ST_K, true);
        const int64_t kdim = x_kdim(L.precision, plen, L.ncol);
        slab_gemm(L, true, X, Xlo, X, Xlo, nao, kdim, Kpart + sl * slab_part, s);
        pr.mark(ST_K, false);
    }
    pr.mark(ST_KREDUCE, true);
    const int nlower = L.ntile * (L.ntile + 1) / 2;
    hipLaunchKernelGGL(k_k_reduce, dim3(nlower, reduce_chunks(L.ktile)), dim3(256), 0, s, Kpart, (int)(L.nslab * L.nsplit_k),
                       L.ntile, L.ktile, nao, 2.0, D, K, Epart);
    hipLaunchKernelGGL(k_energies, dim3(1), dim3(256), 0, s, cvec, ld, Epart, (int64_t)nlower * reduce_chunks(L.ktile), -0.25,
                       E);
    pr.mark(ST_KREDUCE, false);
    pr.mark(ST_BUILD, false);
}

}  // namespace dfjk
