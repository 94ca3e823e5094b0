// Four-centre direct J/K on gfx950: exact (unfitted) Coulomb and exchange
// from Schwarz-screened two-electron integrals over shell quartets, the
// direct-SCF path the package began with (paper, Introduction; "Limitations
// and Future Development: Direct SCF & Other Integral Schemes").  The paper's
// kernels use Rys quadrature; here the integrals are McMurchie-Davidson on
// the Hermite tables the three-centre kernels already use, in the split that
// gives a J-engine for Coulomb:
//
//   (ab|cd) = pref sum_h E^{ab}_f[h] sum_k (-1)^{|k|} E^{cd}_g[k] R_{h+k}(alpha, P - Q),
//   pref = 2 pi^{5/2} / (p q sqrt(p+q)),  alpha = p q / (p+q).
//
// Work split.  Every unordered combination of two pairs is visited once.  A
// workgroup holds one pair u = (a, b) of the class of higher angular momentum, the
// same for all its lanes (its tables are scalar loads), and its lanes walk the
// pairs v = (c, d) of the other class (both sorted by descending Schwarz factor,
// so a wave stops at the first step whose leading v fails Q_u Q_v >= threshold, and
// lanes whose own bound fails sit out).  With u and v of one class, v <= u.
//
// J.  With the densities in Hermite form, Dh_v[h] = w sum_f E_f[h] D_f and, signed,
// Dh_u[k] = w (-1)^{|k|} sum_g E_g[k] D_g (w = 2 for two different shells: both orders
// of the pair), a quartet adds pref sum_h R_{h+k} Dh_v[h] to the Hermite J vector of u,
// which a lane keeps in registers over its walk, and pref sum_k R_{h+k} Dh_u[k] to
// that of v, which goes out with FP64 atomics (adjacent lanes, adjacent addresses);
// J_f = sum_h E_f[h] Jh[h].
//
// K.  K_{mu nu} = sum (mu la|nu si) D_{la si}.  The integrals (ab|cd) give the blocks
// K_ac (with D_bd), K_ad (D_bc), K_bc (D_ad) and K_bd (D_ac), leaving out the
// duplicates of a = b or c = d.  All of them lie in the rows of a and b, which are the
// workgroup's own: they are summed in LDS over the whole walk and added to memory
// once, row by row.  The transposed blocks are the same numbers: the sum F over
// the visits (half of it for u = v) gives K = F + F^T at the end.  The densities come
// from the same rows of D, staged beside them: gathers from memory touch 64 cache
// lines per load, and the heavy launch spent its time there (32 waters: 4.08 ms, 62
// million vector loads; from LDS 2.79 ms, 21 million).
//
// What bounds it: the latency of FP64 chains (Boys function, Hermite recursion) and of
// the table loads at 1 to 3 waves per SIMD, and in the heaviest classes spills ((dd|dd)
// holds 165 values of R, 330 of its 512 registers: 533 stores to and 1,522 loads from
// scratch in its code, (dd|dp) 419 and 472, (dd|pp) 260 and 301; the others save and
// restore registers only); the instructions issued would fill 1.2 ms of the 3.8 ms that
// the three launches take on 32 waters at threshold 1e-10.  Before, every
// ordered combination was visited, in 36 launches, and every quartet added its K blocks
// to memory with scattered FP64 atomics (16 of 31 ms).  Whole builds now against then:
// 3.9 ms against 34, 0.49 against 3.2 for an incremental build of 8 waters; past the sizes
// whose rows fit LDS: 35 waters (D rows of the heavy launch in memory) 4.6 against 34,
// 48 9.0 against 67, 64 17 against 125, 70 (K rows too) 25 against 148.
#include "dfjk_internal.h"
#include "hermite.h"

namespace dfjk {

DirectLayout direct_layout(const Plan &p, bool with_D, bool delta)
{
    DirectLayout L{};
    L.with_D = with_D;
    L.delta = delta;
    size_t off = 0;
    auto take = [&](size_t b) { off = align_up(off, 256); size_t o = off; off += b; return o; };
    L.o_D = (with_D && !delta) ? 0 : take((size_t)p.nao * p.nao * 8);   // D from C, or D - D0
    L.o_dsh = delta ? take(((size_t)p.nsh_ao * p.nsh_ao + 1) * 8) : 0;   // block maxima, then the overall max
    L.o_Dh = take((size_t)std::max<int64_t>(p.dir.herm_total, 1) * 8);
    L.o_Dhv = take((size_t)std::max<int64_t>(p.dir.herm_total, 1) * 8);
    L.o_Jh = take((size_t)std::max<int64_t>(p.dir.herm_total, 1) * 8);
    L.o_Epart = take((size_t)2 * 256 * 8);
    L.bytes = align_up(off, 256);
    return L;
}

// Zeros J, K and the Hermite J vectors.
__global__ __launch_bounds__(256) void k_direct_zero(double *J, double *K, int64_t n, double *Jh, int64_t nh)
{
    const int64_t step = (int64_t)gridDim.x * 256;
    for (int64_t i = blockIdx.x * (int64_t)256 + threadIdx.x; i < 2 * n + nh; i += step) {
        if (i < n) J[i] = 0.0;
        else if (i < 2 * n) K[i - n] = 0.0;
        else Jh[i - 2 * n] = 0.0;
    }
}

// Read of a table entry whose index is the same for every lane of the wave,
// through the constant address space so that it becomes a scalar load (the
// tables are read only for the whole kernel).  Tables written by an earlier
// kernel on the stream are visible: caches are invalidated between kernels.
template <class T>
__device__ __forceinline__ T uniform_load(const T *p)
{
    return *(const __attribute__((address_space(4))) T *)(p);
}

// dD = D - D0, and the largest |dD| over each block of shells (x, y), taken
// over both orientations (the density-weighted Schwarz bound of a quartet).
__global__ void k_dsub(const double *__restrict__ D, const double *__restrict__ D0, int64_t n,
                       double *__restrict__ out)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < n) out[i] = D[i] - D0[i];
}

__global__ void k_shell_dmax(const double *__restrict__ dD, int64_t nao, int32_t nsh, const int32_t *__restrict__ off,
                             double *__restrict__ dsh)
{
    const int64_t xy = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (xy >= (int64_t)nsh * nsh) return;
    const int x = (int)(xy / nsh), y = (int)(xy % nsh);
    double m = 0.0;
    for (int mu = off[x]; mu < off[x + 1]; ++mu)
        for (int nu = off[y]; nu < off[y + 1]; ++nu)
            m = fmax(m, fmax(fabs(dD[(int64_t)mu * nao + nu]), fabs(dD[(int64_t)nu * nao + mu])));
    dsh[xy] = m;
}

// dsh[nsh * nsh] = the largest entry of the table (one block, fixed order).
__global__ __launch_bounds__(256) void k_dmax_all(double *__restrict__ dsh, int64_t n)
{
    __shared__ double red[256];
    double m = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += 256) m = fmax(m, dsh[i]);
    red[threadIdx.x] = m;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + w]);
        __syncthreads();
    }
    if (threadIdx.x == 0) dsh[n] = red[0];
}

// Hermite density of the pairs of one class, entry (h, i), in both layouts: Dh[i][h]
// times (-1)^{|h|} (the pair a workgroup shares) and Dhv[h][i] (a lane's own pair).
template <int LA, int LB>
__device__ __forceinline__ void pair_density(const DirectClassDev &c, const double *__restrict__ D, int64_t nao,
                                             double *__restrict__ Dh, double *__restrict__ Dhv, int64_t t)
{
    constexpr int NA = 2 * LA + 1, NB = 2 * LB + 1, LAB = LA + LB, NH = nherm(LAB);
    const int h = (int)(t / c.npad), i = (int)(t % c.npad);
    if (h >= NH || i >= c.n) return;
    const int oa = c.off_a[i], ob = c.off_b[i];
    const bool same = c.sh_a[i] == c.sh_b[i];
    double s = 0.0;
#pragma unroll
    for (int f = 0; f < NA * NB; ++f) {
        const int ma = f / NB, mb = f % NB;
        const double v = D[(int64_t)(oa + ma) * nao + ob + mb];
        s += c.Eb[(int64_t)(f * NH + h) * c.npad + i] * (same ? v : v + D[(int64_t)(ob + mb) * nao + oa + ma]);
    }
    const int order = h == 0 ? 0 : h < 4 ? 1 : h < 10 ? 2 : h < 20 ? 3 : 4;   // |tuv|: hidx is grouped by it
    Dhv[c.herm_off + t] = s;
    Dh[c.herm_off + (int64_t)i * NH + h] = (order & 1) ? -s : s;
}

// J_f = sum_h E_f[h] Jh[h] of the pairs of one class, entry (f, i), written to both
// triangles (one triangle's positions for a = b: the block holds both).
template <int LA, int LB>
__device__ __forceinline__ void pair_coulomb(const DirectClassDev &c, const double *__restrict__ Jh, int64_t nao,
                                             double *__restrict__ J, int64_t t)
{
    constexpr int NA = 2 * LA + 1, NB = 2 * LB + 1, NH = nherm(LA + LB);
    const int f = (int)(t / c.npad), i = (int)(t % c.npad);
    if (f >= NA * NB || i >= c.n) return;
    double s = 0.0;
#pragma unroll
    for (int h = 0; h < NH; ++h)
        s += c.Eb[(int64_t)(f * NH + h) * c.npad + i] * Jh[c.herm_off + (int64_t)h * c.npad + i];
    const int64_t mu = c.off_a[i] + f / NB, nu = c.off_b[i] + f % NB;
    J[mu * nao + nu] = s;
    if (c.sh_a[i] != c.sh_b[i]) J[nu * nao + mu] = s;
}

// Both passes over every class in one launch: workgroup b belongs to class k for
// start[k] <= b < start[k + 1].
struct PairPass {
    DirectClassDev cls[6];
    uint32_t start[7];
};
template <bool JOUT>
__global__ __launch_bounds__(256) void k_pair_pass(PairPass g, const double *__restrict__ D, int64_t nao,
                                                   double *__restrict__ Dh, double *__restrict__ Dhv,
                                                   const double *__restrict__ Jh, double *__restrict__ J)
{
    int k = 0;
    while (k < 5 && blockIdx.x >= g.start[k + 1]) ++k;
    const DirectClassDev &c = g.cls[k];
    const int64_t t = (int64_t)(blockIdx.x - g.start[k]) * 256 + threadIdx.x;
#define PASS(K, A, B)                                              \
    case K:                                                        \
        if (JOUT) pair_coulomb<A, B>(c, Jh, nao, J, t);            \
        else pair_density<A, B>(c, D, nao, Dh, Dhv, t);            \
        break;
    switch (k) {
        PASS(0, 0, 0) PASS(1, 1, 0) PASS(2, 1, 1) PASS(3, 2, 0) PASS(4, 2, 1) PASS(5, 2, 2)
    }
#undef PASS
}

// Shape of the quartets of u class (LA, LB) and v class (LC, LD).  Light ones: each of
// a workgroup's waves has its own 64 v; every function of v unrolled.  Heavy ones
// (4,000 multiply-adds a quartet and more: long chains on few pairs): four waves
// share 64 v, each with its own copy of R, and are dealt the functions of v.  With the
// line at 6,000, which moves (dp|pp) to the light side, 32 waters take 4.32 ms, not 4.04.
template <int LA, int LB, int LC, int LD>
struct QuartetShape {
    static constexpr int NA = 2 * LA + 1, NB = 2 * LB + 1, NC = 2 * LC + 1, ND = 2 * LD + 1;
    static constexpr int NHU = nherm(LA + LB), NHV = nherm(LC + LD);
    static constexpr int work = NC * ND * NHU * (NHV + NA * NB);
    static constexpr int NS = work < 4000 ? 1 : 4;   // waves that share 64 v
};
constexpr size_t kRowsBytes = 160 * 1024;   // LDS for the rows of a and b (all there is)

// One launch of k_direct: combination k (u class cu[k], v class cv[k]) has the
// workgroups start[k] <= b < start[k + 1]: pieces of vchunk v, for every u.
constexpr int pair_class(int la, int lb) { return la == 0 ? 0 : la == 1 ? 1 + lb : 3 + lb; }
constexpr int kMaxCombos = 13;
struct DirectJob {
    DirectClassDev cls[6];
    uint32_t start[kMaxCombos + 1];
    int32_t vchunk[kMaxCombos], lds[kMaxCombos];
    double tau;
    const double *boys, *D;
    int64_t nao;
    const double *Dh, *Dhv;
    double *Jh, *K;
    const double *dsh;
    int32_t nsh;
};

// The quartets of one combination, as a function of its own: inlined side by side in
// one kernel, the compiler loses the tables' uniformity and spills thousands of
// registers.  A callee's arguments arrive in vector registers, hence the readfirstlanes;
// the job is read where the launch put it, not from a copy in scratch.
typedef const __attribute__((address_space(4))) DirectJob *JobPtr;
typedef __attribute__((address_space(3))) double *LdsPtr;
template <int LA, int LB, int LC, int LD, int WAVES, bool DLDS>
__device__ __noinline__ void direct_quartets(JobPtr job_, int u_, int piece_, int k_, uint32_t lds_)
{
    const uint64_t jp = (uint64_t)job_;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)jp), hi = __builtin_amdgcn_readfirstlane((uint32_t)(jp >> 32));
    const JobPtr jobp = (JobPtr)(((uint64_t)hi << 32) | lo);
    const int u = __builtin_amdgcn_readfirstlane(u_), piece = __builtin_amdgcn_readfirstlane(piece_), kk = __builtin_amdgcn_readfirstlane(k_);
    const LdsPtr rows = (LdsPtr)(uint32_t)__builtin_amdgcn_readfirstlane(lds_);   // K rows of a, then of b
    const __attribute__((address_space(4))) DirectJob &job = *jobp;
    const __attribute__((address_space(4))) DirectClassDev &U = job.cls[pair_class(LA, LB)], &V = job.cls[pair_class(LC, LD)];
    const int vchunk = job.vchunk[kk], rows_in_lds = job.lds[kk];
    using S = QuartetShape<LA, LB, LC, LD>;
    constexpr int NA = S::NA, NB = S::NB, NC = S::NC, ND = S::ND, NHU = S::NHU, NHV = S::NHV;
    constexpr int LU = LA + LB, LV = LC + LD, L = LU + LV, NS = S::NS, G = WAVES / NS;
    constexpr bool same = LA == LC && LB == LD;
    const double tau = job.tau, *__restrict__ boys_tab = job.boys, *__restrict__ D = job.D;
    const double *__restrict__ Dh = job.Dh, *__restrict__ Dhv = job.Dhv, *__restrict__ dsh = job.dsh;
    double *__restrict__ Jh = job.Jh, *__restrict__ K = job.K;
    const int64_t nao = job.nao;
    const int nsh = job.nsh;
    const int nv = same ? u + 1 : V.n;
    const int v0 = piece * vchunk, v1 = min(nv, v0 + vchunk);
    if (v0 >= v1) return;
    const double qu = uniform_load(U.q + u);
    // the Schwarz bound of the walk's end: Q_u Q_v, times the largest |D - D0|
    // anywhere for an incremental build
    const double qwalk = qu * (dsh ? uniform_load(dsh + (int64_t)nsh * nsh) : 1.0);
    if (!(uniform_load(V.q + v0) * qwalk >= tau)) return;
    const int oa = uniform_load(U.off_a + u), ob = uniform_load(U.off_b + u);
    const int sa = uniform_load(U.sh_a + u), sb = uniform_load(U.sh_b + u);
    const bool ab_same = sa == sb;
    const int nao32 = (int)nao, nrows = (ab_same ? NA : NA + NB) * nao32;
    const int brow = ab_same ? 0 : NA;
    const LdsPtr drows = rows + (NA + NB) * nao32;   // D rows of a, then (if another shell) of b
    if (DLDS || rows_in_lds) {
        for (int i = threadIdx.x; i < nrows; i += 64 * WAVES) rows[i] = 0.0;
        if constexpr (DLDS)
            for (int r = 0; r < (ab_same ? NA : NA + NB); ++r)
                for (int i = threadIdx.x; i < nao32; i += 64 * WAVES)
                    drows[r * nao32 + i] = D[(int64_t)(r < NA ? oa + r : ob + r - NA) * nao + i];
        __syncthreads();
    }
    // F[row][col] += x, row = a function of a (0 ..) or of b (NA ..)
    auto add = [&](int row, int col, double x) {
        if (DLDS || rows_in_lds)
            __hip_atomic_fetch_add(rows + (row * nao32 + col), x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        else
            unsafeAtomicAdd(&K[(int64_t)(row < NA ? oa + row : ob + row - NA) * nao + col], x);
    };

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int part = wave % NS, group = wave / NS;
    const double q = uniform_load(U.p + u);
    const double Qx = uniform_load(U.px + u), Qy = uniform_load(U.py + u), Qz = uniform_load(U.pz + u);
    const double *ek = U.Ek + (int64_t)u * (NA * NB * NHU);   // [g][k], signed
    const double *du = Dh + U.herm_off + (int64_t)u * NHU;
    // D between a function of a (row < NA) or b and function col of v
    auto dens = [&](int row, int col) -> double {
        if constexpr (DLDS) return drows[(row < NA ? row : brow + row - NA) * nao32 + col];
        return D[(int64_t)(row < NA ? oa + row : ob + row - NA) * nao + col];
    };
    double ju[NHU];
#pragma unroll
    for (int k = 0; k < NHU; ++k) ju[k] = 0.0;

    for (int jb = v0 + 64 * group; jb < v1; jb += 64 * G) {
        if (!(uniform_load(V.q + jb) * qwalk >= tau)) break;   // the first v of a step is its largest
        const int j = jb + lane;
        if (!(j < v1 && qu * V.q[j] >= tau)) continue;
        const int sc = V.sh_a[j], sd = V.sh_b[j];
        if (dsh) {
            // density-weighted bound: Q_u Q_v times the largest |dD| of the blocks
            // this quartet contracts with (cd and ab for J; bd, bc, ad, ac for K)
            auto m = [&](int x, int y) { return dsh[(int64_t)x * nsh + y]; };
            const double dm = fmax(fmax(fmax(m(sc, sd), m(sa, sb)), fmax(m(sb, sd), m(sb, sc))),
                                   fmax(m(sa, sd), m(sa, sc)));
            if (!(qu * V.q[j] * dm >= tau)) continue;
        }
        const bool cd_same = sc == sd, uv_same = same && j == u;
        const double p = V.p[j];
        const double X = V.px[j] - Qx, Y = V.py[j] - Qy, Z = V.pz[j] - Qz;
        const double pq = p + q, alpha = p * q / pq;
        double F[L + 1];
        boys<L>(alpha * (X * X + Y * Y + Z * Z), F, boys_tab);
        double R[nherm(L)];
        hermite_R<L>(alpha, X, Y, Z, F, R);
        const double pref = kTwoPi52 / (p * q * sqrt(pq));

        // Coulomb, both ways
        // (by the part with the fewest functions: by the first 3.82 ms instead of 3.65, 0.51 instead of 0.49)
        if (NS == 1 || part == NS - 1) {
#pragma unroll
            for (int t = 0; t <= LV; ++t)
#pragma unroll
                for (int x = 0; x + t <= LV; ++x)
#pragma unroll
                    for (int y = 0; y + x + t <= LV; ++y) {
                        const int h = hidx(t, x, y);
                        const double dv = pref * Dhv[V.herm_off + (int64_t)h * V.npad + j];
                        double s = 0.0;
#pragma unroll
                        for (int t2 = 0; t2 <= LU; ++t2)
#pragma unroll
                            for (int x2 = 0; x2 + t2 <= LU; ++x2)
#pragma unroll
                                for (int y2 = 0; y2 + x2 + t2 <= LU; ++y2) {
                                    const int k = hidx(t2, x2, y2);
                                    const double r = R[hidx(t + t2, x + x2, y + y2)];
                                    ju[k] += r * dv;
                                    s += r * uniform_load(du + k);
                                }
                        if (!uv_same) unsafeAtomicAdd(&Jh[V.herm_off + (int64_t)h * V.npad + j], pref * s);
                    }
        }

        // Exchange: function f = (mc, md) of v against every (ma, mb) of u
        const double kpref = uv_same ? 0.5 * pref : pref;
        const int oc = V.off_a[j], od = V.off_b[j];
        auto integrals = [&](int f, double (&I)[NA * NB]) {
            double W[NHU];
#pragma unroll
            for (int k = 0; k < NHU; ++k) W[k] = 0.0;
#pragma unroll
            for (int t = 0; t <= LV; ++t)
#pragma unroll
                for (int x = 0; x + t <= LV; ++x)
#pragma unroll
                    for (int y = 0; y + x + t <= LV; ++y) {
                        const double e = V.Eb[(int64_t)(f * NHV + hidx(t, x, y)) * V.npad + j];
#pragma unroll
                        for (int t2 = 0; t2 <= LU; ++t2)
#pragma unroll
                            for (int x2 = 0; x2 + t2 <= LU; ++x2)
#pragma unroll
                                for (int y2 = 0; y2 + x2 + t2 <= LU; ++y2)
                                    W[hidx(t2, x2, y2)] += e * R[hidx(t + t2, x + x2, y + y2)];
                    }
#pragma unroll
            for (int g = 0; g < NA * NB; ++g) {
                double s = 0.0;
#pragma unroll
                for (int k = 0; k < NHU; ++k) s += uniform_load(ek + g * NHU + k) * W[k];
                I[g] = kpref * s;
            }
        };
        // contributions of one f to the columns c (kc) and d (kd): rows of a, then of b
        auto contract = [&](const double (&I)[NA * NB], int c, int d, double (&kc)[NA + NB], double (&kd)[NA + NB]) {
            double dac[NA], dad[NA], dbc[NB], dbd[NB];
#pragma unroll
            for (int m = 0; m < NA; ++m) { dac[m] = dens(m, c); dad[m] = dens(m, d); }
#pragma unroll
            for (int m = 0; m < NB; ++m) { dbc[m] = dens(NA + m, c); dbd[m] = dens(NA + m, d); }
#pragma unroll
            for (int ma = 0; ma < NA; ++ma)
#pragma unroll
                for (int mb = 0; mb < NB; ++mb) {
                    const double v = I[ma * NB + mb];
                    kc[ma] += v * dbd[mb];
                    kd[ma] += v * dbc[mb];
                    kc[NA + mb] += v * dad[ma];
                    kd[NA + mb] += v * dac[ma];
                }
        };
        auto flush = [&](const double (&x)[NA + NB], int col) {
#pragma unroll
            for (int m = 0; m < NA; ++m) add(m, col, x[m]);
            if (!ab_same)
#pragma unroll
                for (int m = NA; m < NA + NB; ++m) add(m, col, x[m]);
        };
        if constexpr (NS == 1) {
            double kd[ND][NA + NB];
#pragma unroll
            for (int md = 0; md < ND; ++md)
#pragma unroll
                for (int m = 0; m < NA + NB; ++m) kd[md][m] = 0.0;
#pragma unroll
            for (int mc = 0; mc < NC; ++mc) {
                double kc[NA + NB];
#pragma unroll
                for (int m = 0; m < NA + NB; ++m) kc[m] = 0.0;
#pragma unroll
                for (int md = 0; md < ND; ++md) {
                    double I[NA * NB];
                    integrals(mc * ND + md, I);
                    contract(I, oc + mc, od + md, kc, kd[md]);
                }
                flush(kc, oc + mc);
            }
            if (!cd_same)
#pragma unroll
                for (int md = 0; md < ND; ++md) flush(kd[md], od + md);
        } else {
#pragma unroll 1
            for (int f = part; f < NC * ND; f += NS) {
                double I[NA * NB], kc[NA + NB], kd[NA + NB];
#pragma unroll
                for (int m = 0; m < NA + NB; ++m) kc[m] = kd[m] = 0.0;
                integrals(f, I);
                contract(I, oc + f / ND, od + f % ND, kc, kd);
                flush(kc, oc + f / ND);
                if (!cd_same) flush(kd, od + f % ND);
            }
        }
    }

    // Hermite J of u: over the wave, then one atomic per entry and wave
    if (NS == 1 || part == NS - 1) {
#pragma unroll
        for (int t = 0; t <= LU; ++t)
#pragma unroll
            for (int x = 0; x + t <= LU; ++x)
#pragma unroll
                for (int y = 0; y + x + t <= LU; ++y) {
                    const int k = hidx(t, x, y);
                    double s = ju[k];
#pragma unroll
                    for (int w = 32; w > 0; w >>= 1) s += __shfl_xor(s, w);
                    if (lane == 0 && s != 0.0)
                        unsafeAtomicAdd(&Jh[U.herm_off + (int64_t)k * U.npad + u], ((t + x + y) & 1) ? -s : s);
                }
    }
    if (DLDS || rows_in_lds) {
        __syncthreads();
        for (int i = threadIdx.x; i < nrows; i += 64 * WAVES) {
            const double x = rows[i];
            if (x != 0.0) {
                const int r = i / nao32, col = i - r * nao32;
                unsafeAtomicAdd(&K[(int64_t)(r < NA ? oa + r : ob + r - NA) * nao + col], x);
            }
        }
    }
}

// The combinations by the registers they take, heaviest first within a launch: one
// launch each for those of up to 512 (one wave per SIMD, workgroups of 4 waves), up to
// 256 (2, 8 waves) and up to 168 (3, 6 waves).  Classes of one launch run side by
// side: one launch per combination took 1.20 ms instead of 0.54 for the incremental build
// of 8 waters.  Squeezing (dp|dp) and lighter ones of the first launch into 256 registers,
// for a second wave, makes them spill too: 4.31 ms instead of 3.82 on 32 waters.  The row counts
// keep two sets of rows (K and D) in LDS up to 1,024, 1,280 and 2,560 AO; beyond, K alone
// up to twice that, and then neither.
#define COMBOS_0(X) X(0, 2, 2, 2, 2) X(1, 2, 2, 2, 1) X(2, 2, 1, 2, 1) X(3, 2, 2, 1, 1) X(4, 2, 2, 2, 0)       \
                    X(5, 2, 1, 1, 1) X(6, 2, 1, 2, 0) X(7, 2, 2, 1, 0) X(8, 1, 1, 1, 1) X(9, 2, 0, 1, 1)       \
                    X(10, 2, 1, 1, 0) X(11, 2, 0, 2, 0) X(12, 2, 2, 0, 0)
#define COMBOS_1(X) X(0, 2, 1, 0, 0) X(1, 1, 1, 1, 0) X(2, 2, 0, 1, 0) X(3, 1, 1, 0, 0) X(4, 2, 0, 0, 0)
#define COMBOS_2(X) X(0, 1, 0, 1, 0) X(1, 1, 0, 0, 0) X(2, 0, 0, 0, 0)
constexpr int group_waves(int group) { return group == 0 ? 4 : group == 1 ? 8 : 6; }
constexpr int group_rows(int group) { return group == 0 ? 10 : group == 1 ? 8 : 4; }   // most rows of a and b
constexpr int group_simd(int group) { return group == 2 ? 3 : group + 1; }             // waves per SIMD

template <int GROUP, bool DLDS>
__global__ __launch_bounds__(64 * group_waves(GROUP), group_simd(GROUP)) void k_direct(DirectJob job)
{
    extern __shared__ double rows[];
    uint32_t lds = (uint32_t)(uintptr_t)(LdsPtr)rows;
    asm volatile("" : "+s"(lds));   // opaque: the callees take the address from here, not from the compiler's tables
    const JobPtr args = (JobPtr)__builtin_amdgcn_kernarg_segment_ptr();   // job itself: the only argument
    int k = 0;
    while (k < kMaxCombos - 1 && blockIdx.x >= job.start[k + 1]) ++k;
    const int local = (int)(blockIdx.x - job.start[k]);
#define RUN(I, A, B, C, E)                                                                                    \
    case I: {                                                                                                 \
        const int n = job.cls[pair_class(A, B)].n;                                                            \
        direct_quartets<A, B, C, E, group_waves(GROUP), DLDS>(args, local % n, local / n, I, lds);                                      \
        break;                                                                                                \
    }
    if constexpr (GROUP == 0) {
        switch (k) { COMBOS_0(RUN) }
    } else if constexpr (GROUP == 1) {
        switch (k) { COMBOS_1(RUN) }
    } else {
        switch (k) { COMBOS_2(RUN) }
    }
#undef RUN
}

// Symmetrise J (mean of the two triangles), K = F + F^T, add the reference J0, K0
// of an incremental build, and form the block partials of sum D.J and sum D.K
// over the lower triangle mu >= nu.
__global__ __launch_bounds__(256) void k_direct_finish(int64_t nao, const double *__restrict__ D, const double *__restrict__ J0,
                                                       const double *__restrict__ K0, double *__restrict__ J,
                                                       double *__restrict__ K, double *__restrict__ Epart)
{
    const int64_t ntri = nao * (nao + 1) / 2;
    double ej = 0.0, ek = 0.0;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < ntri; e += (int64_t)gridDim.x * blockDim.x) {
        int64_t mu = (int64_t)((sqrt(8.0 * (double)e + 1.0) - 1.0) * 0.5);
        while (mu * (mu + 1) / 2 > e) --mu;
        while ((mu + 1) * (mu + 2) / 2 <= e) ++mu;
        const int64_t nu = e - mu * (mu + 1) / 2;
        const int64_t a = mu * nao + nu, b = nu * nao + mu;
        double jv = mu == nu ? J[a] : 0.5 * (J[a] + J[b]);
        double kv = K[a] + K[b];
        if (J0) { jv += J0[a]; kv += K0[a]; }   // increment on top of the reference (symmetric) J0, K0
        J[a] = jv; J[b] = jv;
        K[a] = kv; K[b] = kv;
        const double dw = mu == nu ? D[a] : D[a] + D[b];
        ej += dw * jv;
        ek += dw * kv;
    }
    __shared__ double sj[256], sk[256];
    sj[threadIdx.x] = ej; sk[threadIdx.x] = ek;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) { sj[threadIdx.x] += sj[threadIdx.x + w]; sk[threadIdx.x] += sk[threadIdx.x + w]; }
        __syncthreads();
    }
    if (threadIdx.x == 0) { Epart[blockIdx.x] = sj[0]; Epart[256 + blockIdx.x] = sk[0]; }
}

// E_J = 1/2 sum D.J, E_K = -1/4 sum D.K from the 256 block partials, in a fixed order.
__global__ __launch_bounds__(256) void k_direct_energy(const double *__restrict__ Epart, double *__restrict__ E)
{
    __shared__ double sj[256], sk[256];
    sj[threadIdx.x] = Epart[threadIdx.x]; sk[threadIdx.x] = Epart[256 + threadIdx.x];
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) { sj[threadIdx.x] += sj[threadIdx.x + w]; sk[threadIdx.x] += sk[threadIdx.x + w]; }
        __syncthreads();
    }
    if (threadIdx.x == 0) { E[0] = 0.5 * sj[0]; E[1] = -0.25 * sk[0]; }
}

// The walk over v is cut where a combination has fewer than kMinWalks u: a workgroup
// costs the staging and the flush of its rows, so longer walks win (cut for 2,048
// workgroups 5.35 ms, 512: 4.04, 256: 3.89, 128: 3.82 on 32 waters; 8 waters 0.54, 0.54,
// 0.53, 0.51).
constexpr int kMinWalks = 128;

template <int LA, int LB, int LC, int LD, int WAVES>
static uint32_t plan_combo(DirectJob &g, int k, size_t &lds)
{
    using S = QuartetShape<LA, LB, LC, LD>;
    const DirectClassDev &U = g.cls[pair_class(LA, LB)], &V = g.cls[pair_class(LC, LD)];
    if (U.n <= 0 || V.n <= 0) return 0;
    const int step = 64 * (WAVES / S::NS), steps = (V.n + step - 1) / step;
    const int pieces = std::max(1, std::min(steps, (kMinWalks + U.n - 1) / U.n));
    g.vchunk[k] = (steps + pieces - 1) / pieces * step;
    const size_t bytes = (size_t)(S::NA + S::NB) * (size_t)g.nao * 8;
    g.lds[k] = bytes <= kRowsBytes;
    if (g.lds[k]) lds = std::max(lds, bytes);
    return (uint32_t)U.n * (uint32_t)((V.n + g.vchunk[k] - 1) / g.vchunk[k]);
}

template <int GROUP>
static void launch_group(DirectJob g, hipStream_t s)
{
    size_t lds = 0;
    uint32_t total = 0;
    int n = 0;
#define PLAN(I, A, B, C, E)                          \
    g.start[n++] = total;                            \
    total += plan_combo<A, B, C, E, group_waves(GROUP)>(g, I, lds);
    if constexpr (GROUP == 0) { COMBOS_0(PLAN) }
    else if constexpr (GROUP == 1) { COMBOS_1(PLAN) }
    else { COMBOS_2(PLAN) }
#undef PLAN
    for (; n <= kMaxCombos; ++n) g.start[n] = total;
    if (total == 0) return;
    const size_t both = (size_t)2 * group_rows(GROUP) * (size_t)g.nao * 8;
    if (both <= kRowsBytes)
        hipLaunchKernelGGL((k_direct<GROUP, true>), dim3(total), dim3(64 * group_waves(GROUP)), both, s, g);
    else
        hipLaunchKernelGGL((k_direct<GROUP, false>), dim3(total), dim3(64 * group_waves(GROUP)), lds, s, g);
}

// The Hermite densities (JOUT false) or J (true) of every class.
template <bool JOUT>
static void launch_pair_pass(const DirectClassDev *cls, const double *D, int64_t nao, double *Dh, double *Dhv,
                             const double *Jh, double *J, hipStream_t s)
{
    PairPass g{};
    uint32_t total = 0;
    for (int k = 0; k < 6; ++k) {
        const int la = kPairClassLa[k], lb = kPairClassLb[k];
        const int64_t per = JOUT ? (2 * la + 1) * (2 * lb + 1) : nherm(la + lb);
        g.cls[k] = cls[k];
        g.start[k] = total;
        if (cls[k].n > 0) total += (uint32_t)((per * cls[k].npad + 255) / 256);
    }
    g.start[6] = total;
    if (total > 0)
        hipLaunchKernelGGL(k_pair_pass<JOUT>, dim3(total), dim3(256), 0, s, g, D, nao, Dh, Dhv, Jh, J);
}

void launch_direct_build(const Plan &p, const DirectLayout &L, const double *C, int32_t nocc, const double *Din,
                         const double *D0, const double *J0, const double *K0, double *J, double *K, double *E,
                         char *scratch, hipStream_t s)
{
    const int64_t nao = p.nao;
    const DirectState &ds = p.dir;
    const double *Dfull = Din;
    if (!L.with_D) {
        double *Dw = reinterpret_cast<double *>(scratch + L.o_D);
        launch_density(C, nao, nocc, 2.0, Dw, s);
        Dfull = Dw;
    }
    // the density whose J and K are integrated: D, or dD = D - D0 with the
    // shell-block bound table of the density-weighted screen
    const double *D = Dfull;
    const double *dsh = nullptr;
    if (L.delta) {
        double *dD = reinterpret_cast<double *>(scratch + L.o_D);
        double *tab = reinterpret_cast<double *>(scratch + L.o_dsh);
        hipLaunchKernelGGL(k_dsub, dim3((unsigned)((nao * nao + 255) / 256)), dim3(256), 0, s, Din, D0, nao * nao, dD);
        const int64_t nxy = (int64_t)p.nsh_ao * p.nsh_ao;
        hipLaunchKernelGGL(k_shell_dmax, dim3((unsigned)((nxy + 255) / 256)), dim3(256), 0, s, dD, nao, p.nsh_ao,
                           ds.shell_off, tab);
        hipLaunchKernelGGL(k_dmax_all, dim3(1), dim3(256), 0, s, tab, nxy);
        D = dD;
        dsh = tab;
    }
    double *Dh = reinterpret_cast<double *>(scratch + L.o_Dh);
    double *Dhv = reinterpret_cast<double *>(scratch + L.o_Dhv);
    double *Jh = reinterpret_cast<double *>(scratch + L.o_Jh);
    double *Epart = reinterpret_cast<double *>(scratch + L.o_Epart);
    const int64_t nz = 2 * nao * nao + ds.herm_total;
    hipLaunchKernelGGL(k_direct_zero, dim3((unsigned)std::min<int64_t>((nz + 1023) / 1024, 4096)), dim3(256), 0, s, J,
                       K, nao * nao, Jh, ds.herm_total);
    launch_pair_pass<false>(ds.cls, D, nao, Dh, Dhv, nullptr, nullptr, s);
    DirectJob g{};
    for (int k = 0; k < 6; ++k) g.cls[k] = ds.cls[k];
    g.tau = p.thresh; g.boys = ds.boys; g.D = D; g.nao = nao;
    g.Dh = Dh; g.Dhv = Dhv; g.Jh = Jh; g.K = K; g.dsh = dsh; g.nsh = p.nsh_ao;
    launch_group<0>(g, s);
    launch_group<1>(g, s);
    launch_group<2>(g, s);
    launch_pair_pass<true>(ds.cls, nullptr, nao, nullptr, nullptr, Jh, J, s);
    hipLaunchKernelGGL(k_direct_finish, dim3(256), dim3(256), 0, s, nao, Dfull, L.delta ? J0 : nullptr,
                       L.delta ? K0 : nullptr, J, K, Epart);
    hipLaunchKernelGGL(k_direct_energy, dim3(1), dim3(256), 0, s, Epart, E);
}

}  // namespace dfjk
