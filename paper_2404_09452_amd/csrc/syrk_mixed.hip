// Mixed-precision products for K on gfx950 matrix cores (FP32 is with FP64 in
// syrk_f64.hip):
//   syrk mode:    P = A A^T on the lower tiles      (direct mixed K)
//   general mode: P = A B^T on every tile           (incremental K)
// with split-K into FP64 partial tiles summed elsewhere in a fixed order.
//
//  BF16x3:  every operand x stored as hi + lo, both BF16 (hi = rn(x),
//           lo = rn(x - hi)); a b ~ hi_a hi_b + hi_a lo_b + lo_a hi_b on
//           v_mfma_f32_16x16x32_bf16 (the lo lo term, ~2^-16 relative, is
//           dropped).  Products accumulate in FP32 over at most kChunk k
//           values and are then added into FP64 accumulators.  The k loop is
//           pipelined like the FP64 tile GEMM: the next chunk is prefetched
//           into registers while the current one is consumed from
//           double-buffered LDS, one barrier per chunk.
//  int8:    below.
//
// 16x16x32 bf16 layout (checked on the device): lane l supplies
// A[l%16][8(l/16)..+7], B[8(l/16)..+7][l%16]; accumulator r of lane l is
// D[4(l/16) + r][l%16].
#include "dfjk_internal.h"

#include <algorithm>
#include <vector>

namespace dfjk {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4m __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int T = 128;          // output tile (four waves, 64x64 each)
constexpr int kChunk = 512;     // k values per FP32 accumulation chunk

__device__ __forceinline__ void mixed_tile(int t, bool lower, int ntm, int &tm, int &tn)
{
    if (lower) {
        int r = (int)((sqrt(8.0 * (double)t + 1.0) - 1.0) * 0.5);
        while (r * (r + 1) / 2 > t) --r;
        while ((r + 1) * (r + 2) / 2 <= t) ++r;
        tm = r;
        tn = t - r * (r + 1) / 2;
    } else {
        tm = t % ntm;
        tn = t / ntm;
    }
}

struct MixedArgs {
    const void *A, *Alo, *B, *Blo;   // [M][ld] planes
    int64_t ld;                      // = kdim
    int64_t M;                       // rows of A and of B (nao)
    int64_t kdim, ksplit;
    int ntm;
    int lower;                       // 1: syrk mode (B = A, tiles tn <= tm)
    double *partial;                 // [split][tile][T][T]
};

// Chunk of 32 k; four planes (A hi/lo, B hi/lo) of 128 x 32 bf16.
__global__ __launch_bounds__(256) void k_gemm_bf16x3(MixedArgs g)
{
    constexpr int KC = 32, LDK = KC + 8, NP = 4;
    using Elem = unsigned short;
    __shared__ __attribute__((aligned(16))) Elem sm[2 * NP * T * LDK];   // [buf][plane][T * LDK]

    int tm, tn;
    mixed_tile(blockIdx.x, g.lower, g.ntm, tm, tn);
    const int64_t m0 = (int64_t)tm * T, n0 = (int64_t)tn * T;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wm = wave >> 1, wn = wave & 1;
    const int64_t kb = (int64_t)blockIdx.y * g.ksplit;
    const int64_t ke = min(kb + g.ksplit, g.kdim);

    f64x4m acc[4][4];
    f32x4 a32[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            acc[i][j] = f64x4m{0.0, 0.0, 0.0, 0.0};
            a32[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        }

    // Each thread moves 16-byte pieces: row = idx / (KC*esz/16), column piece idx % (...).
    constexpr int PIECES = KC * (int)sizeof(Elem) / 16;    // 16-byte pieces per row
    constexpr int LOADS = T * PIECES / 256;                // pieces per thread per plane
    uint4 reg[NP][LOADS];
    const Elem *src[NP];
    src[0] = static_cast<const Elem *>(g.A);
    src[1] = static_cast<const Elem *>(g.lower ? g.A : g.B);
    src[2] = static_cast<const Elem *>(g.Alo);
    src[3] = static_cast<const Elem *>(g.lower ? g.Alo : g.Blo);
    auto load = [&](int64_t k0) {
#pragma unroll
        for (int pl = 0; pl < NP; ++pl) {
            const int64_t r0 = (pl == 1 || pl == 3) ? n0 : m0;
#pragma unroll
            for (int it = 0; it < LOADS; ++it) {
                const int idx = tid + 256 * it, row = idx / PIECES, pc = idx % PIECES;
                const int64_t r = r0 + row;
                reg[pl][it] = (r < g.M)
                    ? *reinterpret_cast<const uint4 *>(src[pl] + r * g.ld + k0 + pc * (16 / sizeof(Elem)))
                    : uint4{0, 0, 0, 0};
            }
        }
    };
    auto store = [&](int buf) {
#pragma unroll
        for (int pl = 0; pl < NP; ++pl)
#pragma unroll
            for (int it = 0; it < LOADS; ++it) {
                const int idx = tid + 256 * it, row = idx / PIECES, pc = idx % PIECES;
                *reinterpret_cast<uint4 *>(&sm[((buf * NP + pl) * T + row) * LDK + pc * (16 / sizeof(Elem))]) =
                    reg[pl][it];
            }
    };

    int since = 0;
    if (kb < ke) {
        load(kb);
        store(0);
        __syncthreads();
        int buf = 0;
        for (int64_t k0 = kb; k0 < ke; k0 += KC) {
            const bool more = k0 + KC < ke;
            if (more) load(k0 + KC);
            const unsigned short *P0 = reinterpret_cast<const unsigned short *>(sm) + (buf * 4) * T * LDK;
            const unsigned short *Ah = P0, *Bh = P0 + T * LDK, *Al = P0 + 2 * T * LDK, *Bl = P0 + 3 * T * LDK;
#pragma unroll
            for (int ks = 0; ks < KC / 32; ++ks) {
                bf16x8 ah[4], al[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int o = (wm * 64 + i * 16 + (lane & 15)) * LDK + ks * 32 + 8 * (lane >> 4);
                    ah[i] = *reinterpret_cast<const bf16x8 *>(&Ah[o]);
                    al[i] = *reinterpret_cast<const bf16x8 *>(&Al[o]);
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int o = (wn * 64 + j * 16 + (lane & 15)) * LDK + ks * 32 + 8 * (lane >> 4);
                    const bf16x8 bh = *reinterpret_cast<const bf16x8 *>(&Bh[o]);
                    const bf16x8 bl = *reinterpret_cast<const bf16x8 *>(&Bl[o]);
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        a32[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al[i], bh, a32[i][j], 0, 0, 0);
                        a32[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[i], bl, a32[i][j], 0, 0, 0);
                        a32[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[i], bh, a32[i][j], 0, 0, 0);
                    }
                }
            }
            since += KC;
            if (since >= kChunk || !more) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
#pragma unroll
                        for (int r = 0; r < 4; ++r) acc[i][j][r] += (double)a32[i][j][r];
                        a32[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
                    }
                since = 0;
            }
            if (more) {
                store(buf ^ 1);
                __syncthreads();
                buf ^= 1;
            }
        }
    }
    const int ntiles = g.lower ? g.ntm * (g.ntm + 1) / 2 : g.ntm * g.ntm;
    double *dst = g.partial + ((int64_t)blockIdx.y * ntiles + blockIdx.x) * (int64_t)(T * T);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = wm * 64 + i * 16 + 4 * (lane >> 4) + r;
                const int col = wn * 64 + j * 16 + (lane & 15);
                dst[row * T + col] = acc[i][j][r];
            }
}

// ---------------------------------------------------------------------------
// Int8 slices (DFJK_MIXED_INT8), the Ozaki splitting of floating-point
// products into exact integer ones (Ozaki, Ogita, Oishi & Rump, Numer.
// Algorithms 59, 2012): with x = 2^{e_x} sum_i a_i 2^{-7(i+1)} and y alike,
//   x y ~ 2^{e_x + e_y} sum_{t=0}^{4} 2^{-7(t+2)} sum_{i+j=t} a_i b_j,
// the products of combined order i + j <= 4 (15 of the 25).  Each order t is
// an exact int32 sum on v_mfma_i32_16x16x64_i8 over one scale block (256 k,
// |sum| < 5 * 127 * 127 * 256 < 2^31), then the five orders are combined in
// FP64 and added with the block's scale 2^{e_x + e_y} into FP64
// accumulators.  The only rounding is the truncation of the slices.
//
// DFJK_MIXED_INT8_FAST (FAST below) keeps the orders i + j <= 3 and the one
// order-4 product a_2 b_2 (11 products; slice a_4 is neither stored, loaded nor
// used).  a_2 b_2 stays because on the diagonal it is a square: dropped, it
// would shift every K_mu mu the same way and bias E_K (by 1e-6 Eh already on
// three waters), whereas the other dropped order-4 products carry no sign.
//
// What bounds it: the operand traffic from L2 into LDS.  Without the loads
// the 128 x 64 FAST kernel below runs in 57% of its time; without its LDS reads
// in 88%, without the folds in 91%.  So the loads are shaped first:
//  - a DMA instruction (global_load_lds_dwordx4, 64 lanes x 16 bytes, LDS in
//    lane order) takes consecutive 16-byte pieces of a row's chunk (64 k x NS
//    slices, contiguous in X): 256 bytes of each of 4 rows for FAST.  One
//    slice of 16 rows per instruction (64-byte segments) moved 6.6 TB/s and
//    no more; this shape took 960 AO x 450,560 k from 3.58 to 2.67 ms (128 x 64
//    tiles) and 3,840 x 655,360 from 67.0 to 54.2 ms (int8: 4.47 to 4.06 and
//    84.0 to 76.0 ms).
//  - inside a row the pieces are stored at a permuted slot, so that the 16
//    rows of a fragment read fall on 16 different 16-byte bank groups: slot =
//    piece xor (row mod 16) for the 16 pieces of FAST, (piece + (row / 4) mod 4)
//    mod 20 for the 20 of five slices.
//  - FAST keeps the fragments of the next chunk in a second register set, read
//    while the MFMAs use the current one, with one barrier a chunk; its 128-wide
//    form has three chunk buffers (two chunks in flight).  3,840 AO: 54.2 to
//    49.7 (registers) to 48.4 ms (third buffer).  Five slices leave neither the
//    registers nor the LDS for it: there a chunk is read, the barrier tells
//    that its buffer is free, and the DMA of the chunk two ahead goes into it.
//
// Workgroup: 128 rows x 64 columns of the output (half of a 128 x 128 partial
// tile, blk = 2 tile + half) on eight waves, or (FAST, narrow molecules) a
// 64 x 64 tile on four waves with two workgroups per CU, each wave 2 x 2
// fragments of 16 x 16: five int32 order accumulators (80 registers), FP64
// accumulators (32).
// 16x16x64 i8 layout: lane l supplies row l%16 and 16 consecutive k bytes of
// k group l/16 for both operands; accumulator r of lane l is D[4(l/16)+r][l%16].
typedef int i32x4 __attribute__((ext_vector_type(4)));

// s_waitcnt immediates (gfx9 encoding: vmcnt bits 3:0 and 15:14, expcnt
// 6:4, lgkmcnt 11:8; a field at its maximum does not wait).  Issued through
// the builtin so the compiler's own wait insertion knows what has retired.
constexpr int i8_wait_vm(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8); }
constexpr int i8_wait_vm_lgkm0(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4); }
constexpr int kWaitLgkm0 = 15 | (7 << 4) | (0 << 8) | (3 << 14);  // lgkmcnt(0)

struct I8Args {
    const unsigned char *A, *B;   // [M][kdim / 64][NS][64] slices
    const double *sA, *sB;        // [M][kdim / 256] block scales
    int64_t kdim, M, ksplit;      // ksplit: a multiple of kI8Block
    int ntm;
    int lower;
    int nsplit;
    double *partial;              // [split][tile][TM][TM]
};

// TM x 64 outputs (TM = 128: half of a 128-wide tile; 64: a whole tile) on
// waves of 32 x 32.
template <int TM, bool FAST>
__device__ __forceinline__ void gemm_i8_tile(I8Args g, unsigned blk)
{
    constexpr int WGN = 2, WGM = TM / 32, NW = WGM * WGN, RB = 2, CB = 2;
    constexpr bool HALF = TM == 128;
    static_assert(TM == 128 || (TM == 64 && FAST), "64-wide tiles are FAST only");
    constexpr int AR = TM, BR = 64;                                      // rows of the two operands
    constexpr int NS = FAST ? kI8Slices - 1 : kI8Slices;                 // slices stored and loaded
    constexpr int NP = NS * kI8Chunk / 16, PITCH = NP * 16;              // 16-byte pieces and bytes of a row's chunk
    constexpr int NF = (AR + BR) * NP / 64, NFA = AR * NP / 64;          // DMA instructions per chunk, those of A
    constexpr int NFW = (NF + NW - 1) / NW, NFS = NFW * NW;              // per wave; slots incl. spares
    constexpr int NBUF = FAST && HALF ? 3 : 2;
    static_assert(AR * NP % 64 == 0 && (AR + BR) * NP % 64 == 0, "whole DMA instructions per operand");
    // chunk buffers as separate arrays: the compiler can then tell a read of
    // one from a DMA into another (which buffer is known at compile time
    // below) and does not wait for unrelated loads
    __shared__ __attribute__((aligned(1024))) unsigned char sm0[NFS * 1024];
    __shared__ __attribute__((aligned(1024))) unsigned char sm1[NFS * 1024];
    __shared__ __attribute__((aligned(1024))) unsigned char sm2[NBUF == 3 ? NFS * 1024 : 16];

    // workgroup -> (split, tile, half).  With a split count that is a multiple
    // of the XCD count, XCD x (workgroups are dispatched round-robin over the
    // XCDs) runs whole splits x, x + 8, ..., so each XCD's L2 holds one k
    // range of X for every tile of a split.
    const int nt = g.lower ? g.ntm * (g.ntm + 1) / 2 : g.ntm * g.ntm;   // tiles per split
    const int nth = HALF ? 2 * nt : nt;                                  // workgroups per split
    int split, th;
    if (g.nsplit % kXcds == 0) {
        const int xcd = blk % kXcds, local = blk / kXcds;
        split = xcd + kXcds * (local / nth);
        th = local % nth;
    } else {
        split = blk / nth;
        th = blk % nth;
    }
    const int half = HALF ? th & 1 : 0, tile = HALF ? th >> 1 : th;
    int tm, tn;
    mixed_tile(tile, g.lower, g.ntm, tm, tn);
    const int64_t m0 = (int64_t)tm * TM, n0 = (int64_t)tn * TM + 64 * half;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave / WGN, wn = wave % WGN;
    const int64_t kb = (int64_t)split * g.ksplit;
    const int64_t ke = min(kb + g.ksplit, g.kdim);
    const int64_t rowb = g.kdim * NS;                 // bytes per row
    const int64_t nblk = g.kdim / kI8Block;

    // this lane's byte offset for each DMA instruction of its wave, relative to
    // the first row of the operand's TM-row tile (which is < M); rows past
    // M read row M-1, whose products only reach outputs that are dropped.
    // Spare slots repeat the last instruction's loads.  The host keeps 128
    // rows below 4 GiB.
    const int64_t a0 = m0, b0 = (int64_t)tn * TM;
    uint32_t loff[NFW];
#pragma unroll
    for (int q = 0; q < NFW; ++q) {
        const int piece = min(wave + NW * q, NF - 1) * 64 + lane, row = piece / NP, slot = piece % NP;
        const int p = FAST ? slot ^ (row & 15) : (slot - ((row >> 2) & 3) + NP) % NP;
        const bool isA = row < AR;
        const int64_t r = min(isA ? m0 + row : n0 + row - AR, g.M - 1);
        loff[q] = (uint32_t)((r - (isA ? a0 : b0)) * rowb + 16 * p);
    }
    auto load = [&](int64_t k0, unsigned char *dstbuf) {
        const int64_t cb = (k0 / kI8Chunk) * PITCH;
#pragma unroll
        for (int q = 0; q < NFW; ++q) {
            const int f = wave + NW * q;
            const unsigned char *base = (min(f, NF - 1) < NFA ? g.A + a0 * rowb : g.B + b0 * rowb) + cb;
            __builtin_amdgcn_global_load_lds((const void *)(base + loff[q]),
                                             (__attribute__((address_space(3))) void *)(dstbuf + f * 1024), 16,
                                             0, 0);
        }
    };
    // fragments of one chunk: lane l of slice s reads piece 4 s + l/16 of row l%16
    const int fr = lane & 15, kg = lane >> 4;
    auto frags = [&](const unsigned char *cur, i32x4 (&af)[NS][RB], i32x4 (&bf)[NS][CB]) {
        const unsigned char *Ra = cur + wm * RB * 16 * PITCH, *Rb = cur + (AR + wn * CB * 16) * PITCH;
#pragma unroll
        for (int sl = 0; sl < NS; ++sl) {
            const int p = 4 * sl + kg, slot = FAST ? p ^ fr : (p + (fr >> 2)) % NP, off = fr * PITCH + slot * 16;
#pragma unroll
            for (int j = 0; j < CB; ++j) bf[sl][j] = *reinterpret_cast<const i32x4 *>(Rb + j * 16 * PITCH + off);
#pragma unroll
            for (int i = 0; i < RB; ++i) af[sl][i] = *reinterpret_cast<const i32x4 *>(Ra + i * 16 * PITCH + off);
        }
    };

    double acc[RB][CB][4];
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int j = 0; j < CB; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.0;
    i32x4 lev[kI8Slices][RB][CB];   // order sums t = 0..4 of the current block
    auto products = [&](const i32x4 (&af)[NS][RB], const i32x4 (&bf)[NS][CB], bool start) {
#pragma unroll
        for (int si = 0; si < NS; ++si)
#pragma unroll
            for (int sj = 0; sj < NS; ++sj)
#pragma unroll
                for (int i = 0; i < RB; ++i)
#pragma unroll
                    for (int j = 0; j < CB; ++j) {
                        const bool kept = FAST ? si + sj <= 3 || (si == 2 && sj == 2) : si + sj <= 4;
                        if (!kept) continue;
                        // the first product of each order sum in a block starts it from zero
                        const bool first = start && si == (FAST && si + sj == 4 ? 2 : 0);
                        const i32x4 cin = first ? i32x4{0, 0, 0, 0} : lev[si + sj][i][j];
                        lev[si + sj][i][j] =
                            __builtin_amdgcn_mfma_i32_16x16x64_i8(af[si][i], bf[sj][j], cin, 0, 0, 0);
                    }
    };

    // Block scales of the operand rows, staged through LDS one block ahead:
    // thread t < AR + BR loads its row's scale of the next block into a
    // register during a block and writes it to ssc[next % 2] at the start of
    // the next block, at least three barriers before the fold of that block
    // reads it.
    __shared__ double ssc[2][AR + BR];
    const int64_t srow_t = tid < AR ? m0 + tid : n0 + (tid - AR);
    const double *sbase_t = tid < AR ? g.sA : g.sB;
    const bool sown = tid < AR + BR && srow_t < g.M;
    double snext = 0.0;
    auto scale_fetch = [&](int64_t b) { snext = (sown && b < nblk) ? sbase_t[srow_t * nblk + b] : 0.0; };
    // FP64 fold of a block: sum_t 2^{-7t} (order t sum) times the block scales.
    // The sums of orders 1 and 2, and of 3 and 4, are joined in int32 first
    // (|128 S_1 + S_2| < 2^30, |128 S_3 + S_4| < 2^30: five conversions and
    // FMAs become three, same value).
    auto fold = [&](const double *sc) {
        double sb[CB];
#pragma unroll
        for (int j = 0; j < CB; ++j) sb[j] = sc[AR + (wn * CB + j) * 16 + fr] * 0x1p-14;
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            double sa[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) sa[r] = sc[(wm * RB + i) * 16 + 4 * kg + r];
#pragma unroll
            for (int j = 0; j < CB; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int s12 = lev[1][i][j][r] * 128 + lev[2][i][j][r];
                    const int s34 = lev[3][i][j][r] * 128 + lev[4][i][j][r];
                    const double v = fma(fma((double)s34, 0x1p-14, (double)s12), 0x1p-14, (double)lev[0][i][j][r]);
                    acc[i][j][r] = fma(v, sa[r] * sb[j], acc[i][j][r]);
                }
        }
    };

    // One scale block per iteration: four chunks whose five order sums live
    // only inside the iteration (the first chunk starts them from zero), then
    // their FP64 fold.  Every chunk step issues one DMA (past the end: the
    // last chunk again, never read), so each wait keeps a known number of a
    // wave's loads in flight (they retire in order; the scale loads among
    // them only make a wait stricter).  Barriers without memory fences keep
    // those loads outstanding across them.
    const int64_t nch = (ke - kb) / kI8Chunk;
    auto chunk_k = [&](int64_t ci) { return kb + min(ci, nch - 1) * kI8Chunk; };
    if (kb < ke) {
        scale_fetch(kb / kI8Block);
        load(chunk_k(0), sm0);
        load(chunk_k(1), sm1);
        if constexpr (NBUF == 3) load(chunk_k(2), sm2);
        __builtin_amdgcn_s_waitcnt(i8_wait_vm((NBUF - 1) * NFW));
        __builtin_amdgcn_s_barrier();
        if constexpr (FAST) {
            // step c: this wave's fragments of chunk c are (or are arriving) in
            // registers and chunk c + 1 has landed once only NBUF - 2 newer
            // chunks are outstanding; the barrier makes both true for every
            // wave, so chunk c's buffer takes the DMA of chunk c + NBUF, the
            // fragments of c + 1 are read and the MFMAs run on chunk c
            i32x4 af0[NS][RB], bf0[NS][CB], af1[NS][RB], bf1[NS][CB];
            frags(sm0, af0, bf0);
            auto step = [&](int64_t ci, int c, unsigned char *cur, const unsigned char *nxt, i32x4 (&af)[NS][RB],
                            i32x4 (&bf)[NS][CB], i32x4 (&afn)[NS][RB], i32x4 (&bfn)[NS][CB], int64_t blkn) {
                __builtin_amdgcn_s_waitcnt(i8_wait_vm_lgkm0((NBUF - 2) * NFW));
                __builtin_amdgcn_s_barrier();
                load(chunk_k(ci + NBUF), cur);
                if (c == 0) scale_fetch(blkn);
                __builtin_amdgcn_sched_barrier(0);
                frags(nxt, afn, bfn);
                products(af, bf, c == 0);
                __builtin_amdgcn_sched_barrier(0);
            };
            // a block whose first chunk lies in p0 and its next ones in p1, p2 (NBUF = 2: p0 again)
            auto block = [&](int64_t k0, unsigned char *p0, unsigned char *p1, unsigned char *p2) {
                const int64_t b = k0 / kI8Block, ci = (k0 - kb) / kI8Chunk;
                if (tid < AR + BR) ssc[b & 1][tid] = snext;
                unsigned char *p3 = NBUF == 3 ? p0 : p1;
                step(ci, 0, p0, p1, af0, bf0, af1, bf1, b + 1);
                step(ci + 1, 1, p1, p2, af1, bf1, af0, bf0, b + 1);
                step(ci + 2, 2, p2, p3, af0, bf0, af1, bf1, b + 1);
                step(ci + 3, 3, p3, NBUF == 3 ? p1 : p0, af1, bf1, af0, bf0, b + 1);
                fold(ssc[b & 1]);
            };
            if constexpr (NBUF == 3) {
                for (int64_t k0 = kb;;) {
                    block(k0, sm0, sm1, sm2);
                    if ((k0 += kI8Block) >= ke) break;
                    block(k0, sm1, sm2, sm0);
                    if ((k0 += kI8Block) >= ke) break;
                    block(k0, sm2, sm0, sm1);
                    if ((k0 += kI8Block) >= ke) break;
                }
            } else {
                for (int64_t k0 = kb; k0 < ke; k0 += kI8Block) block(k0, sm0, sm1, sm0);
            }
        } else {
            // a chunk's fragments are read from LDS into registers first, then
            // (after a barrier: every wave has read that buffer) the DMA of the
            // chunk two ahead goes into the same buffer, then the MFMAs run
            for (int64_t k0 = kb; k0 < ke; k0 += kI8Block) {
                const int64_t b = k0 / kI8Block;
                if (tid < AR + BR) ssc[b & 1][tid] = snext;
                scale_fetch(b + 1);
#pragma unroll
                for (int c = 0; c < kI8Block / kI8Chunk; ++c) {
                    const int64_t ci = (k0 - kb) / kI8Chunk + c;     // chunk index in this split (ci % 2 == c % 2)
                    unsigned char *cur = (c & 1) ? sm1 : sm0;
                    i32x4 af[NS][RB], bf[NS][CB];
                    frags(cur, af, bf);
                    __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
                    __builtin_amdgcn_s_barrier();
                    load(chunk_k(ci + 2), cur);
                    __builtin_amdgcn_sched_barrier(0);   // the DMA goes out before the MFMAs
                    products(af, bf, c == 0);
                    __builtin_amdgcn_sched_barrier(0);   // and the wait stays after them
                    __builtin_amdgcn_s_waitcnt(i8_wait_vm(NFW));
                    __builtin_amdgcn_s_barrier();
                }
                fold(ssc[b & 1]);
            }
        }
        __builtin_amdgcn_s_waitcnt(i8_wait_vm(0));   // no DMA into LDS outlives the workgroup
    }
    double *dst = g.partial + ((int64_t)split * nt + tile) * (int64_t)(TM * TM) + 64 * half;
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int j = 0; j < CB; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = (wm * RB + i) * 16 + 4 * kg + r;
                const int col = (wn * CB + j) * 16 + fr;
                dst[row * TM + col] = acc[i][j][r];
            }
}

constexpr int i8_threads(int TM) { return 4 * TM; }   // one wave per 32 x 32 outputs

template <int TM, bool FAST>
__global__ __launch_bounds__(i8_threads(TM)) __attribute__((amdgpu_waves_per_eu(2, 2)))
void k_gemm_i8(I8Args g)
{
    gemm_i8_tile<TM, FAST>(g, blockIdx.x);
}

// The int8 K of several molecules in one launch (batches): workgroup b runs
// workgroup b - blk_start[m] of molecule m's own launch, descriptors by value.
constexpr int kI8GroupMax = 16;
struct I8Group {
    int32_t n;
    uint32_t blk_start[kI8GroupMax + 1];
    I8Args g[kI8GroupMax];
};
static_assert(sizeof(I8Group) <= 4096, "kernel arguments are limited to 4 KB");

template <int TM, bool FAST>
__global__ __launch_bounds__(i8_threads(TM)) __attribute__((amdgpu_waves_per_eu(2, 2)))
void k_gemm_i8_group(I8Group grp)
{
    int m = 0;
    while (m + 1 < grp.n && blockIdx.x >= grp.blk_start[m + 1]) ++m;
    gemm_i8_tile<TM, FAST>(grp.g[m], blockIdx.x - grp.blk_start[m]);
}

// Tile of the int8_fast K: 64-wide (two workgroups per CU, less above the
// diagonal or past nao, a third more operand traffic) up to 1,440 AO, where
// both reach 170 TFLOP/s FP64-equivalent; 480 AO 158.8 against 141.5, 960 AO 195
// against 164, 1,200 AO 180 against 167, but 1,920 AO 151 against 193 and 3,840
// AO 139 against 200 (the best split count of each).
int i8_fast_tile(int64_t nao) { return nao <= 1440 ? 64 : T; }

// Split count of the int8 K.  64-wide tiles: the largest multiple of the XCD
// count up to 64 (128 above 960 AO: short k ranges keep a split's panels in L2) of
// at least four scale blocks each, within 5% of the fewest rounds of the chip
// (960 AO, 16 / 24 / 32 / 64 splits: 2.42 / 2.34 / 2.19 / 2.13 ms; 1,440 AO, 32 /
// 64 / 128: 15.3 / 13.5 / 12.2 ms), or of the best multiple where that is within 30%:
// whole splits per XCD count for more than even rounds (whole builds of 390 / 420 / 510 /
// 570 / 690 AO with 18 / 54 / 28 / 45 / 62 splits 0.380 / 0.488 / 0.823 / 1.01 / 2.08 ms, with
// 16 / 32 / 56 / 64 / 64 0.341 / 0.434 / 0.719 / 0.884 / 1.90).  128-wide tiles (half a tile per workgroup,
// one per CU), all with the same k length: the time is (rounds of workgroups) x
// (k per split); counts that are multiples of the XCD count run whole splits per
// XCD (rounds counted per XCD), smaller k lengths fall back to any count.
int i8_nsplit(int64_t nao, int64_t kdim, bool lower, int tile, int num_cus)
{
    const int ntm = (int)((nao + tile - 1) / tile);
    const int64_t nt = lower ? ntm * (ntm + 1) / 2 : ntm * ntm;
    const int64_t wg = tile == T ? 2 * nt : nt;
    const int slots = (num_cus > 0 ? num_cus : 256) * (tile == T ? 1 : 2);
    const int xslots = std::max(1, slots / kXcds);
    const int64_t nblk = kdim / kI8Block;
    const int most = tile == T || nao <= 960 ? 64 : 128;
    const int maxs = (int)std::max<int64_t>(1, std::min<int64_t>(most, nblk / 4));
    std::vector<double> cost(maxs + 1, 1e300);
    double best = 1e300;
    for (int ns = 1; ns <= maxs; ++ns) {
        const int64_t per = (nblk + ns - 1) / ns;
        const int64_t rounds = ns % kXcds == 0 ? (wg * (ns / kXcds) + xslots - 1) / xslots
                                               : (wg * ns + slots - 1) / slots;
        cost[ns] = (double)rounds * (double)per;
        best = std::min(best, cost[ns]);
    }
    if (tile != T) {
        for (int ns = maxs / kXcds * kXcds; ns > 0; ns -= kXcds)
            if (cost[ns] <= 1.05 * best) return ns;
        double whole = 1e300;
        for (int ns = kXcds; ns <= maxs; ns += kXcds) whole = std::min(whole, cost[ns]);
        if (whole <= 1.3 * best)
            for (int ns = maxs / kXcds * kXcds; ns > 0; ns -= kXcds)
                if (cost[ns] <= 1.05 * whole) return ns;
        for (int ns = maxs; ns > 1; --ns)
            if (cost[ns] <= 1.05 * best) return ns;
        return 1;
    }
    // a split count that is a multiple of the XCD count runs whole splits per
    // XCD, so the tiles of one k range share their panels in one L2 while
    // they run together: the cheapest such count is taken when within 15% of
    // the best and a split's workgroups fill at most four rounds of one XCD
    // (32-water cluster, 72 workgroups per split: 7 splits in turn 9.2-9.5 ms
    // per build, 8 / 16 / 32 / 64 whole splits per XCD 9.76 / 9.22 / 8.97 /
    // 9.05 ms; 128-water cluster, 930 per split: 3 splits in turn 1.15 s, 8
    // per XCD 1.21 s)
    int bx = 0;
    if (wg <= 4 * xslots)
        for (int ns = kXcds; ns <= maxs; ns += kXcds)
            if (bx == 0 || cost[ns] < cost[bx]) bx = ns;
    if (bx > 0 && cost[bx] <= 1.15 * best) return bx;
    // else the fewest splits within 7% of the best (int8_fast, 1,920 AO: 1 / 2 /
    // 16 splits 34.5 / 35.6 / 38.2 ms; 3,840 AO: 3 / 5 / 8 splits 67.7 / 69.6 / 74.3 ms)
    for (int ns = 1; ns <= maxs; ++ns)
        if (cost[ns] <= 1.07 * best) return ns;
    return 1;
}

static I8Args i8_args(const void *A, const double *sA, const void *B, const double *sB, int64_t nao, int64_t kdim,
                      bool lower, int nsplit, int tile, double *part)
{
    I8Args g{};
    g.A = static_cast<const unsigned char *>(A);
    g.B = static_cast<const unsigned char *>(B);
    g.sA = sA; g.sB = sB;
    g.kdim = kdim; g.M = nao;
    g.ntm = (int)((nao + tile - 1) / tile);
    g.lower = lower ? 1 : 0;
    g.ksplit = ((kdim / kI8Block) + nsplit - 1) / nsplit * kI8Block;
    g.partial = part;
    g.nsplit = nsplit;
    return g;
}
static int64_t i8_workgroups(const I8Args &g, int tile)
{
    return (tile == T ? 2 : 1) * (int64_t)(g.lower ? g.ntm * (g.ntm + 1) / 2 : g.ntm * g.ntm) * g.nsplit;
}

// Split-K partial tiles (tile wide: 128, or 64 for fast) of A B^T.
void launch_gemm_i8(bool lower, const void *A, const double *sA, const void *B, const double *sB, int64_t nao,
                    int64_t kdim, int nsplit, bool fast, int tile, double *part, hipStream_t s)
{
    const I8Args g = i8_args(A, sA, B, sB, nao, kdim, lower, nsplit, tile, part);
    const dim3 grid((unsigned)i8_workgroups(g, tile)), block(i8_threads(tile));
    if (!fast) hipLaunchKernelGGL((k_gemm_i8<T, false>), grid, block, 0, s, g);
    else if (tile == T) hipLaunchKernelGGL((k_gemm_i8<T, true>), grid, block, 0, s, g);
    else hipLaunchKernelGGL((k_gemm_i8<64, true>), grid, block, 0, s, g);
}

// Lower-tile int8 K partials of several molecules (one X and its block
// scales each, kdim[i] long, nsplit[i] splits), all on tiles of one width, as
// launch_gemm_i8 lays them out, in launches of up to kI8GroupMax molecules.
void launch_gemm_i8_group(bool fast, int tile, int n, const void *const *X, const double *const *sX,
                          const int64_t *nao, const int64_t *kdim, const int *nsplit, double *const *part,
                          hipStream_t s)
{
    I8Group grp{};
    int64_t total = 0;
    const dim3 block(i8_threads(tile));
    auto flush = [&]() {
        if (grp.n == 0) return;
        grp.blk_start[grp.n] = (uint32_t)total;
        const dim3 grid((unsigned)total);
        if (!fast) hipLaunchKernelGGL((k_gemm_i8_group<T, false>), grid, block, 0, s, grp);
        else if (tile == T) hipLaunchKernelGGL((k_gemm_i8_group<T, true>), grid, block, 0, s, grp);
        else hipLaunchKernelGGL((k_gemm_i8_group<64, true>), grid, block, 0, s, grp);
        grp = I8Group{};
        total = 0;
    };
    for (int i = 0; i < n; ++i) {
        const I8Args g = i8_args(X[i], sX[i], X[i], sX[i], nao[i], kdim[i], true, nsplit[i], tile, part[i]);
        const int64_t nwg = i8_workgroups(g, tile);
        if (nwg <= 0) continue;
        if (grp.n == kI8GroupMax || total + nwg > (int64_t)UINT32_MAX / 2) flush();
        grp.blk_start[grp.n] = (uint32_t)total;
        grp.g[grp.n++] = g;
        total += nwg;
    }
    flush();
}

// Split count: one round of workgroups (two per CU), each split a multiple
// of the chunk of the precision and at least 512 k long.
static int mixed_splits(int ntiles, int64_t kdim, int num_cus)
{
    const int slots = 2 * (num_cus > 0 ? num_cus : 256);
    int ns = ntiles >= slots ? 1 : slots / ntiles;
    const int64_t maxs = kdim / 512;
    if (ns > maxs) ns = (int)(maxs > 0 ? maxs : 1);
    return ns < 1 ? 1 : ns;
}

int mixed_nsplit(int64_t nao, int64_t kdim, bool lower, int num_cus)
{
    const int ntm = (int)((nao + T - 1) / T);
    return mixed_splits(lower ? ntm * (ntm + 1) / 2 : ntm * ntm, kdim, num_cus);
}

void launch_gemm_bf16x3(bool lower, const void *A, const void *Alo, const void *B, const void *Blo, int64_t nao,
                        int64_t kdim, int nsplit, double *part, hipStream_t s)
{
    MixedArgs g{};
    g.A = A; g.Alo = Alo; g.B = B; g.Blo = Blo;
    g.ld = kdim; g.M = nao; g.kdim = kdim;
    g.ntm = (int)((nao + T - 1) / T);
    g.lower = lower ? 1 : 0;
    g.ksplit = (int64_t)align_up((size_t)((kdim + nsplit - 1) / nsplit), 32);
    g.partial = part;
    const int ntiles = lower ? g.ntm * (g.ntm + 1) / 2 : g.ntm * g.ntm;
    hipLaunchKernelGGL(k_gemm_bf16x3, dim3(ntiles, nsplit), dim3(256), 0, s, g);
}

}  // namespace dfjk
