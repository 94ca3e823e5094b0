// FP64 and FP32 K contraction with operands moved by LDS DMA: the split-K
// partial tiles of C = A B^T (A, B: rows of the half-transformed tensor, k
// contiguous), lower tiles only for K = X X^T or every tile for the
// increment's X1 X2^T.  Partial tiles are FP64; FP32 products accumulate in
// FP32 over at most 512 k, then go into FP64 accumulators, so FP32 rounding
// does not grow with the contraction length.
//
// Workgroup: one T x T tile of one k split; v_mfma_f64_16x16x4f64 or
// v_mfma_f32_16x16x4f32 (lane l supplies A[l%16][l/16] and B[l/16][l%16];
// accumulator r of lane l is D[l/16 + 4r][l%16] in FP64, D[4(l/16) + r][l%16]
// in FP32).
//
// A chunk is 128 bytes of every operand row (16 k in FP64, 32 in FP32).
// Operands go from global memory straight into LDS (global_load_lds_dwordx4:
// 16 bytes per lane, the lanes of one instruction filling 1 KB in lane order,
// 8 rows each) through a ring of chunk buffers; one barrier per chunk.  Row r
// keeps its 16-byte piece p at slot p xor (r/2 mod 8), so a fragment read of 16
// bytes a lane (piece 4h + l/16 of row l%16) meets each of the 16 bank groups
// once in every 16 lanes.  One read gives a lane 2 (FP64) or 4 (FP32) values, used
// by as many MFMAs.  In FP64 a step then covers k {2g + e} over the lane groups g,
// the same for both operands.  In FP32, where the order of the sums shows in the
// result, X keeps each 16 k transposed as 4 x 4 (f32_k_slot), so that step e covers
// k 4e .. 4e + 3 and the sums run in ascending k.
// Rows past M read row M-1; their products reach only outputs the reduction
// drops.
//
// What bounds it: the FP64 (FP32) matrix pipes.  One wave of each workgroup on
// a SIMD waits at the barrier while another workgroup's wave runs, so small
// buffers (more workgroups per CU) count for more than deep ones: two buffers
// and 16-byte reads against three and 8-byte ones, FP64: 64-wide tiles 6.41 ->
// 6.19 ms (960 AO x 450,560 k, 136 splits), 96-wide 10.0 -> 6.32 ms per build's K
// (two waves per SIMD from two workgroups), 128-wide 184.7 -> 168.0 ms (3,840 AO x
// 778,240 k: 70.6 TFLOP/s executed; a large library FP64 GEMM reaches 71.5),
// whitening of 61,440 x 2,816 rows 7.78 -> 7.01 ms.  FP32 against the
// register-staged GEMM it replaced: 720 AO x 261,120 k 1.95 -> 1.42 ms.
#include "dfjk_internal.h"

#include <algorithm>
#include <type_traits>

namespace dfjk {

namespace {

constexpr int kRowBytes = 128;       // bytes of an operand row per chunk
constexpr int kFoldChunks = 16;      // FP32: chunks (512 k) between folds into FP64

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

struct SyrkArgs {
    const void *A, *B;               // [M][ld], [N][ld] rows, k contiguous
    int64_t ld, M, N;
    int64_t kdim, ksplit, ksub;      // ranges of ksplit k, each cut in nsub parts of ksub (multiples of the chunk)
    int ntm, ntn;                    // tiles along M and N
    int lower;                       // 1: tiles with tn <= tm (K = X X^T), else every tile
    int tri_k;                       // 1: B(n, k) = 0 for k > n, so a tile stops at its last column
    int nsplit, nsub;                // nsplit counts the parts
    double *partial;                 // [split][tile][T][T], or
    double *C;                       // C[m][n] (ldc) when partial is null (FP64)
    int64_t ldc;
};

// Waves, chunk buffers and waves per SIMD of each (type, tile).
template <class E, int T> struct SyrkShape {
    static constexpr bool f64 = std::is_same<E, double>::value;
    static constexpr int WGM = f64 && T == 128 ? 4 : 2, WGN = 2;
    static constexpr int NBUF = f64 || T == 128 ? 2 : 3;
    static constexpr int EU = f64 ? (T == 96 ? 2 : 4) : (T == 64 ? 3 : 2);
    static constexpr int threads = 64 * WGM * WGN;
};

// s_waitcnt immediates (gfx9: vmcnt bits 3:0 and 15:14, expcnt 6:4, lgkmcnt
// 11:8; a field at its maximum does not wait)
template <int N> constexpr int wait_vm() { return (N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8); }

// Workgroup `blk` of a launch over g (ntiles x nsplit workgroups).  EDGES (lower
// tiles only): a wave leaves out the MFMAs of its 16 x 16 fragments above the
// diagonal or past the last row, in a k loop of its own (a test in the common
// loop cost full tiles 14%), and the sub-tile a wave takes rotates over the
// workgroups so that the idle ones spread over the SIMDs.
template <class E, int T, bool EDGES>
__device__ __forceinline__ void syrk_tile(SyrkArgs g, unsigned blk)
{
    using S = SyrkShape<E, T>;
    constexpr int WGM = S::WGM, WGN = S::WGN, NW = WGM * WGN, NBUF = S::NBUF;
    constexpr int WTM = T / WGM, WTN = T / WGN, MB = WTM / 16, NB = WTN / 16;
    constexpr int KC = kRowBytes / (int)sizeof(E);
    constexpr int OPB = T * kRowBytes;               // bytes of one operand's chunk
    constexpr int NI = 2 * T / 8;                    // DMA instructions per chunk (8 rows each)
    constexpr int NIW = NI / NW;                     // per wave
    static_assert(NIW * NW == NI && NIW * NBUF <= 60, "DMA instructions must spread evenly over the waves");
    // separate arrays: the compiler can tell a read of one from a DMA into another
    __shared__ __attribute__((aligned(1024))) char s0[2 * OPB];
    __shared__ __attribute__((aligned(1024))) char s1[2 * OPB];
    __shared__ __attribute__((aligned(1024))) char s2[NBUF == 3 ? 2 * OPB : 16];

    const int ntiles = g.lower ? g.ntm * (g.ntm + 1) / 2 : g.ntm * g.ntn;
    // workgroup -> (split, tile), 1-D grid.  With a split count that is a
    // multiple of the XCD count, XCD x (workgroups go round-robin over the
    // XCDs) runs whole splits x, x + 8, ...: the tiles of one k range share
    // their panels in one L2 instead of every L2 fetching every panel.
    int tile, split;
    if (g.nsplit % kXcds == 0) {
        const int xcd = blk % kXcds, local = blk / kXcds;
        split = xcd + kXcds * (local / ntiles);
        tile = local % ntiles;
    } else {
        split = blk / ntiles;
        tile = blk % ntiles;
    }
    int tm, tn;
    if (g.lower) {
        int r = (int)((sqrt(8.0 * (double)tile + 1.0) - 1.0) * 0.5);
        while (r * (r + 1) / 2 > tile) --r;
        while ((r + 1) * (r + 2) / 2 <= tile) ++r;
        tm = r;
        tn = tile - r * (r + 1) / 2;
    } else {
        tm = tile % g.ntm;
        tn = tile / g.ntm;
        if (g.tri_k) tn = g.ntn - 1 - tn;   // the longest k ranges first
    }
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int sub = EDGES ? (wave + (int)(blk / kXcds)) % NW : wave;
    const int wm = sub / WGN, wn = sub % WGN;
    // a range's parts rotate over its splits: the last one, which may be short, would
    // else be one XCD's in every range (8 parts)
    const int range = split / g.nsub, part = (split + range) % g.nsub;
    const int64_t kr = (int64_t)range * g.ksplit, kb = kr + part * g.ksub;
    int64_t ke = min(min(kb + g.ksub, kr + g.ksplit), g.kdim);
    if (g.tri_k) ke = min(ke, (int64_t)(tn + 1) * T);
    const int nch = (int)((ke - kb) / KC);

    // this lane's source of chunk 0 for each DMA instruction of its wave
    const char *src[NIW];
#pragma unroll
    for (int q = 0; q < NIW; ++q) {
        const int ins = wave * NIW + q;
        const bool isA = ins < NI / 2;
        const int r = (ins % (NI / 2)) * 8 + lane / 8;
        const int p = (lane % 8) ^ ((r >> 1) & 7);
        const int64_t row = isA ? min((int64_t)tm * T + r, g.M - 1) : min((int64_t)tn * T + r, g.N - 1);
        src[q] = static_cast<const char *>(isA ? g.A : g.B) + (row * g.ld + kb) * (int64_t)sizeof(E) + 16 * p;
    }
    auto dma = [&](int c, char *buf) {
        const int64_t o = (int64_t)min(c, nch - 1) * kRowBytes;   // past the end: the last chunk again
#pragma unroll
        for (int q = 0; q < NIW; ++q)
            __builtin_amdgcn_global_load_lds(
                (const void *)(src[q] + o),
                (__attribute__((address_space(3))) void *)(buf + (wave * NIW + q) * 8 * kRowBytes), 16, 0, 0);
    };

    f64x4 acc[MB][NB];
    f32x4 a32[S::f64 ? 1 : MB][S::f64 ? 1 : NB];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            acc[i][j] = f64x4{0.0, 0.0, 0.0, 0.0};
            if constexpr (!S::f64) a32[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    auto fold = [&]() {
        if constexpr (!S::f64) {
#pragma unroll
            for (int i = 0; i < MB; ++i)
#pragma unroll
                for (int j = 0; j < NB; ++j) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[i][j][r] += (double)a32[i][j][r];
                    a32[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
                }
        }
    };

    const int fr = lane & 15, kg = lane >> 4;
    unsigned mask = 0;   // fragments that reach outputs the reduction reads
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const int64_t m = (int64_t)tm * T + wm * WTM + i * 16, n = (int64_t)tn * T + wn * WTN + j * 16;
            if (m < g.M && n <= m) mask |= 1u << (i * NB + j);
        }
    mask = __builtin_amdgcn_readfirstlane(mask);
    constexpr unsigned kAll = (1u << (MB * NB)) - 1;
    auto product = [&](auto a, auto b, int i, int j) {
        if constexpr (S::f64) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc[i][j], 0, 0, 0);
        else a32[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, a32[i][j], 0, 0, 0);
    };
    auto mfma = [&](const char *buf, auto whole) {
        using V = typename std::conditional<S::f64, f64x2, f32x4>::type;
        const char *as = buf + wm * WTM * kRowBytes, *bs = buf + OPB + wn * WTN * kRowBytes;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int off = fr * kRowBytes + (((4 * h + kg) ^ ((fr >> 1) & 7)) << 4);
            V a[MB], b[NB];
#pragma unroll
            for (int i = 0; i < MB; ++i) a[i] = *reinterpret_cast<const V *>(as + i * 16 * kRowBytes + off);
#pragma unroll
            for (int j = 0; j < NB; ++j) b[j] = *reinterpret_cast<const V *>(bs + j * 16 * kRowBytes + off);
            if constexpr (decltype(whole)::value) {
#pragma unroll
                for (int e = 0; e < 16 / (int)sizeof(E); ++e)
#pragma unroll
                    for (int i = 0; i < MB; ++i)
#pragma unroll
                        for (int j = 0; j < NB; ++j) product(a[i][e], b[j][e], i, j);
            } else {
#pragma unroll
                for (int i = 0; i < MB; ++i)
#pragma unroll
                    for (int j = 0; j < NB; ++j)
                        if (mask >> (i * NB + j) & 1)
#pragma unroll
                            for (int e = 0; e < 16 / (int)sizeof(E); ++e) product(a[i][e], b[j][e], i, j);
            }
        }
    };
    // chunk c: its DMA has landed for this wave once only NBUF - 2 newer
    // chunks' loads are outstanding; the barrier makes that true for every
    // wave and tells that chunk c - 1's buffer is read; then the DMA of chunk
    // c + NBUF - 1 goes into that buffer and the MFMAs run on chunk c
    auto step = [&](int c, const char *cur, char *nxt, auto whole) {
        __builtin_amdgcn_s_waitcnt(wait_vm<NIW * (NBUF - 2)>());
        __builtin_amdgcn_s_barrier();
        dma(c + NBUF - 1, nxt);
        __builtin_amdgcn_sched_barrier(0);
        if (decltype(whole)::value || mask != 0) mfma(cur, whole);
        __builtin_amdgcn_sched_barrier(0);
        if (!S::f64 && c % kFoldChunks == kFoldChunks - 1) fold();
    };
    auto loop = [&](auto whole) {
        int c = 0;
        if constexpr (NBUF == 3) {
            for (; c + 3 <= nch; c += 3) {   // whole rounds of the buffers
                step(c, s0, s2, whole);
                step(c + 1, s1, s0, whole);
                step(c + 2, s2, s1, whole);
            }
            if (c < nch) step(c, s0, s2, whole);
            if (c + 1 < nch) step(c + 1, s1, s0, whole);
        } else {
            for (; c + 2 <= nch; c += 2) {
                step(c, s0, s1, whole);
                step(c + 1, s1, s0, whole);
            }
            if (c < nch) step(c, s0, s1, whole);
        }
    };

    if (nch > 0) {
        dma(0, s0);
        if constexpr (NBUF == 3) dma(1, s1);
        if constexpr (EDGES) {   // the waves of a workgroup may take either loop: both meet every barrier
            if (mask == kAll) loop(std::true_type{});
            else loop(std::false_type{});
        } else {
            loop(std::true_type{});
        }
        __builtin_amdgcn_s_waitcnt(wait_vm<0>());   // no DMA into LDS outlives the workgroup
        fold();
    }

    if (g.partial) {
        double *dst = g.partial + ((int64_t)split * ntiles + tile) * (int64_t)(T * T);
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = wm * WTM + i * 16 + (S::f64 ? kg + 4 * r : 4 * kg + r);
                    const int col = wn * WTN + j * 16 + fr;
                    dst[row * T + col] = acc[i][j][r];
                }
        return;
    }
    if constexpr (S::f64) {
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int64_t m = (int64_t)tm * T + wm * WTM + i * 16 + kg + 4 * r;
                    const int64_t n = (int64_t)tn * T + wn * WTN + j * 16 + fr;
                    if (m < g.M && n < g.N) g.C[m * g.ldc + n] = acc[i][j][r];
                }
    }
}

template <class E, int T, bool EDGES>
__global__ __launch_bounds__((SyrkShape<E, T>::threads))
__attribute__((amdgpu_waves_per_eu(SyrkShape<E, T>::EU)))
void k_syrk(SyrkArgs g)
{
    syrk_tile<E, T, EDGES>(g, blockIdx.x);
}

// The K syrk of several molecules in one launch (batches of small
// molecules): workgroup b runs workgroup b - blk_start[m] of molecule m's own
// launch, descriptors by value (no device table, so the launch can be
// captured).  Each molecule's partial tiles are those of its own launch.
constexpr int kSyrkGroupMax = 16;
struct SyrkGroup {
    int32_t n;
    uint32_t blk_start[kSyrkGroupMax + 1];
    SyrkArgs g[kSyrkGroupMax];
};
static_assert(sizeof(SyrkGroup) <= 4096, "kernel arguments are limited to 4 KB");

template <int T>
__global__ __launch_bounds__((SyrkShape<double, T>::threads))
__attribute__((amdgpu_waves_per_eu(SyrkShape<double, T>::EU)))
void k_syrk_f64_group(SyrkGroup grp)
{
    int m = 0;
    while (m + 1 < grp.n && blockIdx.x >= grp.blk_start[m + 1]) ++m;
    syrk_tile<double, T, T == 64>(grp.g[m], blockIdx.x - grp.blk_start[m]);
}

// 64-wide lower tiles leave out edge fragments when whole tiles execute over 10%
// more than whole fragments would, up to 960 AO (FP64: 210 AO 44 -> 41 us, 330 AO
// 170 -> 142 us, 390 AO 284 -> 256 us, 720 AO 2.33 -> 2.17 ms; 960 AO, 5% more: 6.16 ->
// 6.18 ms; 1,440 AO 32.9 -> 35.8 ms).
bool skip_edges(int64_t nao)
{
    const int64_t t = (nao + 63) / 64, f = (nao + 15) / 16;
    return nao <= 960 && t * (t + 1) * 4096 > 1.1 * (double)(f * (f + 1) * 256);
}

template <class E, int T, bool EDGES = false>
void launch_tiles(const SyrkArgs &g, unsigned nwg, hipStream_t s)
{
    hipLaunchKernelGGL((k_syrk<E, T, EDGES>), dim3(nwg), dim3(SyrkShape<E, T>::threads), 0, s, g);
}

// Split-K partial tiles of A B^T (A = B for the lower-tile syrk): M rows of
// kdim, nsplit splits of ksplit (a multiple of the chunk), tiles of T (64, 96 or 128).
template <class E>
void launch_syrk(bool lower, const E *A, const E *B, int64_t M, int64_t kdim, int64_t ksplit, int64_t ksub,
                 int nsplit, int nsub, int T, double *partial, hipStream_t s)
{
    SyrkArgs g{};
    g.A = A; g.B = B; g.ld = kdim; g.M = M; g.N = M; g.kdim = kdim; g.ksplit = ksplit;
    g.ntm = g.ntn = (int)((M + T - 1) / T);
    g.lower = lower ? 1 : 0;
    g.nsplit = nsplit;
    g.ksub = ksub;
    g.nsub = nsub;
    g.partial = partial;
    const int ntiles = lower ? g.ntm * (g.ntm + 1) / 2 : g.ntm * g.ntn;
    if (ntiles <= 0 || nsplit <= 0) return;
    const unsigned nwg = (unsigned)(ntiles * nsplit);
    if (T == 128) launch_tiles<E, 128>(g, nwg, s);
    else if (T == 96) launch_tiles<E, 96>(g, nwg, s);
    else if (lower && skip_edges(M)) launch_tiles<E, 64, true>(g, nwg, s);
    else launch_tiles<E, 64>(g, nwg, s);
}

}  // namespace

void launch_syrk_f64(bool lower, const double *A, const double *B, int64_t M, int64_t kdim, int64_t ksplit,
                     int nsplit, int T, double *partial, hipStream_t s)
{
    launch_syrk<double>(lower, A, B, M, kdim, ksplit, ksplit, nsplit, 1, T, partial, s);
}

// FP32: nsplit / nsub ranges of ksplit k, in each of which the FP32 sums are
// folded every 512 k from its start; the nsub parts of a range (whole 512 k but
// the last) give more workgroups without moving those folds.
void launch_syrk_f32(bool lower, const float *A, const float *B, int64_t M, int64_t kdim, int64_t ksplit, int nsplit,
                     int nsub, int T, double *partial, hipStream_t s)
{
    constexpr int64_t kFold = kFoldChunks * kRowBytes / sizeof(float);
    const int64_t ksub = nsub > 1 ? (int64_t)align_up((size_t)((ksplit + nsub - 1) / nsub), kFold) : ksplit;
    launch_syrk<float>(lower, A, B, M, kdim, ksplit, ksub, nsplit, nsub, T, partial, s);
}

// Output tile of the FP64 and FP32 K (kdim long): the width that executes the fewest
// products (whole tiles, the diagonal ones included) at the rate each reaches, relative
// to 64-wide tiles on few AO.
//
// FP64, from whole builds on every width (480 to 2,160 AO, nao / 30 to nao orbitals; the
// rule's choice is 0.2% slower than the best on average, 4.7% at worst).  Up to 1,440 AO
// 64-wide tiles fall back as the panels of one of their splits, nao x k, outgrow an
// XCD's L2 (4 MB; time on 64-wide over time on 96-wide tiles, with the panels: 750 AO
// 0.97 at 8 MB, 1.03 at 23, 1.08 at 47; 960 AO 0.99 at 5, 1.02 to 1.04 at 25, 1.06 at 76; 1,200
// AO 0.96 at 17, 1.02 at 86), and up to 640 AO they have half the splits.  Above,
// rates in TFLOP/s executed (1,920 / 3,840 AO): 64-wide 65 / 64, 96-wide 71 / 71,
// 128-wide 71 / 71; whole builds on 128-wide tiles gain from 1,800 AO on (1,650 / 1,740 /
// 1,860 / 1,920 / 2,160 AO: 78.6 and 76.0, 96.6 and 96.9, 128.8 and 120.7, 133.6 and
// 127.9, 213 and 203 ms on 96- and 128-wide tiles).
//
// FP32 executed TFLOP/s at 960 / 1,440 / 1,920 / 3,840 AO: 64-wide 121 / 111 / 106 / 103,
// 96-wide 127 / 130 / 121 / 118, 128-wide 132 / 127 / 129 / 123 (the choice within 3%
// of the autotuner's best at 22 of 23 sizes from 420 to 1,560 AO, 4.5% at the other).
static double tile_rate(int T, int64_t nao, int64_t kdim, bool f64, int num_cus)
{
    if (!f64) return T == 64 ? (nao <= 960 ? 1.0 : 0.88) : T == 96 ? 1.03 : 1.05;
    if (nao > 1440) return T == 64 ? 0.92 : T == 96 ? 1.04 : nao <= 1780 ? 1.027 : 1.10;
    const int64_t t = (nao + 63) / 64, slots = (nao <= 640 ? 32 : 64) * (int64_t)(num_cus > 0 ? num_cus : 256);
    const int64_t splits = std::max<int64_t>(1, std::min<int64_t>(slots / (t * (t + 1) / 2), kdim / 512));
    const double panel = 8e-6 * (double)nao * (double)(kdim / splits);
    const double large = std::min(1.0, std::max(0.0, (panel - 14.0) / 22.0));
    if (T == 64) return 1.0;
    return T == 96 ? std::max(1.0 + 0.08 * large, nao <= 640 ? 1.02 : 1.0) : 1.027 + 0.028 * large;
}

int syrk_tile_width(int64_t nao, int64_t kdim, bool f64, int num_cus)
{
    int best = 64;
    double cost = 1e300;
    for (int T : {64, 96, 128}) {
        const double n = (double)((nao + T - 1) / T);
        double c = n * (n + 1) * T * T;
        const double f = (double)((nao + 15) / 16);
        if (T == 64 && skip_edges(nao)) c = std::min(c, 1.14 * f * (f + 1) * 256.0);   // as measured with EDGES
        c /= tile_rate(T, nao, kdim, f64, num_cus);
        if (c < cost) { cost = c; best = T; }
    }
    return best;
}

// Lower-tile syrk partials of several molecules on T-wide tiles (64, 96 or
// 128), up to kSyrkGroupMax per launch: molecule i has M[i] rows of X (A[i], kdim[i]
// long), nsplit[i] splits of ksplit[i] (a multiple of 16) and its partials
// at partial[i], laid out as launch_syrk_f64 lays them out.
void launch_syrk_f64_group(int T, int n, const double *const *A, const int64_t *M, const int64_t *kdim,
                           const int64_t *ksplit, const int *nsplit, double *const *partial, hipStream_t s)
{
    SyrkGroup grp{};
    int64_t total = 0;
    auto flush = [&]() {
        if (grp.n == 0) return;
        grp.blk_start[grp.n] = (uint32_t)total;
        if (T == 128)
            hipLaunchKernelGGL((k_syrk_f64_group<128>), dim3((unsigned)total), dim3(SyrkShape<double, 128>::threads), 0, s, grp);
        else if (T == 96)
            hipLaunchKernelGGL((k_syrk_f64_group<96>), dim3((unsigned)total), dim3(SyrkShape<double, 96>::threads), 0, s, grp);
        else
            hipLaunchKernelGGL((k_syrk_f64_group<64>), dim3((unsigned)total), dim3(SyrkShape<double, 64>::threads), 0, s, grp);
        grp = SyrkGroup{};
        total = 0;
    };
    for (int i = 0; i < n; ++i) {
        SyrkArgs g{};
        g.A = A[i]; g.B = A[i]; g.ld = kdim[i]; g.M = M[i]; g.N = M[i]; g.kdim = kdim[i]; g.ksplit = g.ksub = ksplit[i]; g.nsub = 1;
        g.ntm = g.ntn = (int)((M[i] + T - 1) / T);
        g.lower = 1;
        g.nsplit = nsplit[i];
        g.partial = partial[i];
        const int64_t nwg = (int64_t)g.ntm * (g.ntm + 1) / 2 * nsplit[i];
        if (nwg <= 0) continue;
        if (grp.n == kSyrkGroupMax || total + nwg > (int64_t)UINT32_MAX / 2) flush();
        grp.blk_start[grp.n] = (uint32_t)total;
        grp.g[grp.n++] = g;
        total += nwg;
    }
    flush();
}

// C = A B^T with B lower triangular in (n, k) (B(n, k) = 0 for k > n), both
// row-major over ld = k: the whitening B_fP = sum_{Q <= P} U_fQ Linv_PQ.  M
// rows of A, N rows of B (a multiple of 128), no split.  128-wide tiles, 64-wide
// ones where those would be fewer than four a CU (4 waters: 228 workgroups whose k
// differs threefold take 54 us, 912 small ones 27).
void launch_gemm_nt_tri(const double *A, const double *B, double *C, int64_t M, int64_t N, int64_t ld,
                        hipStream_t s)
{
    SyrkArgs g{};
    g.A = A; g.B = B; g.ld = ld; g.M = M; g.N = N; g.kdim = ld; g.ksplit = g.ksub = ld; g.nsub = 1;
    const int T = ((M + 127) / 128) * (N / 128) < 1024 ? 64 : 128;
    g.ntm = (int)((M + T - 1) / T);
    g.ntn = (int)((N + T - 1) / T);
    g.lower = 0; g.tri_k = 1; g.nsplit = 1;
    g.C = C; g.ldc = ld;
    const int ntiles = g.ntm * g.ntn;
    if (ntiles <= 0) return;
    if (T == 64) launch_tiles<double, 64>(g, (unsigned)ntiles, s);
    else launch_tiles<double, 128>(g, (unsigned)ntiles, s);
}

}  // namespace dfjk
