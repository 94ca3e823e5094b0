// Host runtime and C ABI of the DF-J/K library: validation, host preparation
// of the shell tables, Schwarz-screening compaction, workspace carving and
// the ordering of the kernel launches.  No kernels live here.
#include <algorithm>
#include <climits>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <initializer_list>
#include <mutex>
#include <numeric>
#include <tuple>
#include <type_traits>
#include <vector>

#include "dfjk_internal.h"

struct dfjk_plan {
    dfjk::Plan p;
};

namespace dfjk {

static thread_local std::string g_last_error;

static int fail(int code, const std::string &msg)
{
    g_last_error = msg;
    return code;
}

#define HIP_OR_FAIL(expr)                                                                        \
    do {                                                                                         \
        hipError_t e_ = (expr);                                                                  \
        if (e_ != hipSuccess)                                                                    \
            return fail(DFJK_E_DEVICE, std::string(#expr) + ": " + hipGetErrorString(e_));      \
    } while (0)

// ---------------------------------------------------------------------------
// Tables generated by the library.

static double binom(int n, int k)
{
    if (k < 0 || k > n) return 0.0;
    double r = 1.0;
    for (int i = 1; i <= k; ++i) r = r * (n - k + i) / i;
    return r;
}

static int cart_index_of(int l, int lx, int ly)
{
    int k = 0;
    for (int x = l; x >= 0; --x)
        for (int y = l - x; y >= 0; --y) {
            if (x == lx && y == ly) return k;
            ++k;
        }
    return -1;
}

// General real solid harmonics in Racah normalisation (Helgaker, Jorgensen,
// Olsen, Molecular Electronic-Structure Theory, eqs. 6.4.47-6.4.50):
// S_lm = N_lm sum_{t,u,v} C_tuv x^{2t+|m|-2(u+v)} y^{2(u+v)} z^{l-2t-|m|},
// C_tuv = (-1)^{t+v-v_m} 4^{-t} (l t)(l-t |m|+t)(t u)(|m| 2v),
// N_lm = sqrt(2 (l+|m|)! (l-|m|)! / 2^{delta_m0}) / (2^{|m|} l!),
// v_m = 0 for m >= 0 and 1/2 for m < 0 (v then runs over half integers).
// m order: p as (x, y, z) = (1, -1, 0); d and f as m = -l..l.
void solid_harmonic_table(double coef[kMaxLAux + 1][7][10])
{
    std::memset(coef, 0, sizeof(double) * (kMaxLAux + 1) * 70);
    auto fact = [](int n) { double r = 1; for (int i = 2; i <= n; ++i) r *= i; return r; };
    for (int l = 0; l <= kMaxLAux; ++l) {
        for (int idx = 0; idx < 2 * l + 1; ++idx) {
            int m;
            if (l == 1) m = (idx == 0) ? 1 : (idx == 1 ? -1 : 0);
            else m = idx - l;
            const int am = std::abs(m);
            const double Nlm = std::sqrt(2.0 * fact(l + am) * fact(l - am) / (m == 0 ? 2.0 : 1.0)) /
                               (std::pow(2.0, am) * fact(l));
            // work with twice v so half-integers are integers: vv = 2v
            const int vv_m = (m < 0) ? 1 : 0;
            for (int t = 0; t <= (l - am) / 2; ++t)
                for (int u = 0; u <= t; ++u) {
                    // v from v_m to floor(|m|/2 - v_m) + v_m, step 1 -> vv step 2
                    const int vmax2 = 2 * (int)std::floor(am / 2.0 - vv_m / 2.0) + vv_m;
                    for (int vv = vv_m; vv <= vmax2; vv += 2) {
                        const int sgn_exp = t + (vv - vv_m) / 2;
                        const double c = ((sgn_exp & 1) ? -1.0 : 1.0) * std::pow(0.25, t) * binom(l, t) *
                                         binom(l - t, am + t) * binom(t, u) * binom(am, vv);
                        const int px = 2 * t + am - 2 * u - vv, py = 2 * u + vv, pz = l - 2 * t - am;
                        coef[l][idx][cart_index_of(l, px, py)] += Nlm * c;
                        (void)pz;
                    }
                }
        }
    }
}

double shell_norm(int l, double a)
{
    // <phi|phi> = (4 pi/(2l+1)) Gamma(l+3/2) / (2 (2a)^{l+3/2}) for Racah-normalised S_lm
    const double val = 4.0 * M_PI / (2 * l + 1) * std::tgamma(l + 1.5) / (2.0 * std::pow(2.0 * a, l + 1.5));
    return 1.0 / std::sqrt(val);
}

// Gauss-Legendre nodes/weights on [-1, 1] (Newton on P_n, long double).
static void gauss_legendre(int n, std::vector<long double> &x, std::vector<long double> &w)
{
    x.assign(n, 0.0L);
    w.assign(n, 0.0L);
    const long double pi = 3.141592653589793238462643383279502884L;
    for (int i = 0; i < (n + 1) / 2; ++i) {
        long double z = cosl(pi * (i + 0.75L) / (n + 0.5L)), pp = 0.0L;
        for (int it = 0; it < 100; ++it) {
            long double p1 = 1.0L, p2 = 0.0L;
            for (int j = 1; j <= n; ++j) {
                const long double p3 = p2;
                p2 = p1;
                p1 = ((2 * j - 1) * z * p2 - (j - 1) * p3) / j;
            }
            pp = n * (z * p1 - p2) / (z * z - 1.0L);
            const long double dz = p1 / pp;
            z -= dz;
            if (fabsl(dz) < 1e-21L) break;
        }
        x[i] = -z;
        x[n - 1 - i] = z;
        w[i] = w[n - 1 - i] = 2.0L / ((1.0L - z * z) * pp * pp);
    }
}

// F_m(T) = int_0^1 t^{2m} exp(-T t^2) dt by 8 panels of 48-point Gauss-Legendre.
const std::vector<double> &boys_table()
{
    static std::vector<double> tab;
    static std::once_flag once;
    std::call_once(once, [] {
        std::vector<long double> gx, gw;
        gauss_legendre(48, gx, gw);
        const int npanel = 8;
        tab.assign((size_t)kBoysNT * kBoysNM, 0.0);
        for (int k = 0; k < kBoysNT; ++k) {
            const long double T = (long double)k * (long double)kBoysH;
            std::vector<long double> acc(kBoysNM, 0.0L);
            for (int pnl = 0; pnl < npanel; ++pnl) {
                const long double a = (long double)pnl / npanel, b = (long double)(pnl + 1) / npanel;
                for (size_t q = 0; q < gx.size(); ++q) {
                    const long double t = 0.5L * (b - a) * gx[q] + 0.5L * (a + b);
                    const long double wt = 0.5L * (b - a) * gw[q] * expl(-T * t * t);
                    long double tp = 1.0L;
                    for (int m = 0; m < kBoysNM; ++m) {
                        acc[m] += wt * tp;
                        tp *= t * t;
                    }
                }
            }
            for (int m = 0; m < kBoysNM; ++m) tab[(size_t)k * kBoysNM + m] = (double)acc[m];
        }
    });
    return tab;
}

Error ensure_device_constants(int device, const double **boys_dev)
{
    static std::mutex mu;
    static const double *addr[256] = {};
    std::lock_guard<std::mutex> lock(mu);
    if (device < 0 || device >= 256) return {DFJK_E_DEVICE, "device index out of range"};
    if (!addr[device]) {
        double coef[kMaxLAux + 1][7][10];
        solid_harmonic_table(coef);
        upload_constants(coef, nullptr);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return {DFJK_E_DEVICE, std::string("constant upload: ") + hipGetErrorString(e)};
        const std::vector<double> &tab = boys_table();
        upload_boys_table(tab.data(), tab.size(), &addr[device], &e);
        if (e != hipSuccess) return {DFJK_E_DEVICE, std::string("Boys table upload: ") + hipGetErrorString(e)};
    }
    *boys_dev = addr[device];
    return {DFJK_OK, ""};
}

void Profiler::mark(int stage, bool begin)
{
    if (!on) return;
    size_t rec;
    if (begin) {
        if (open[stage] >= 0) return;   // already open: stages do not nest with themselves
        rec = rec_stage.size();
        rec_stage.push_back(stage);
        open[stage] = (int)rec;
    } else {
        if (open[stage] < 0) return;    // unmatched end
        rec = (size_t)open[stage];
        open[stage] = -1;
    }
    const size_t idx = 2 * rec + (begin ? 0 : 1);
    while (pool.size() <= idx) {
        hipEvent_t e{};
        if (hipEventCreate(&e) != hipSuccess) { on = false; return; }
        pool.push_back(e);
    }
    (void)hipEventRecord(pool[idx], stream);
}

static const char *kStageNames[ST_COUNT] = {
    "setup.int3c", "setup.metric", "setup.cholesky", "setup.inverse", "setup.whiten",
    "build.density", "build.J", "build.halftransform", "build.K", "build.Kreduce_energies", "span.build",
    "span.setup"};

static int check_device(int *device)
{
    int n = 0;
    if (hipGetDeviceCount(&n) != hipSuccess || n <= 0) {
        (void)hipGetLastError();
        return fail(DFJK_E_NO_DEVICE, "no GPU device is visible");
    }
    HIP_OR_FAIL(hipGetDevice(device));
    return DFJK_OK;
}

// ---------------------------------------------------------------------------
// Plan creation (host only).

static int validate_basis(const dfjk_basis *b, int natm, int lmax, const char *name)
{
    if (!b) return fail(DFJK_E_INVALID, std::string(name) + " basis is NULL");
    if (b->nshell <= 0) return fail(DFJK_E_INVALID, std::string(name) + " basis has no shells");
    if (!b->shell_atom || !b->shell_l || !b->shell_exp)
        return fail(DFJK_E_INVALID, std::string(name) + " basis has a NULL array");
    for (int i = 0; i < b->nshell; ++i) {
        if (b->shell_atom[i] < 0 || b->shell_atom[i] >= natm)
            return fail(DFJK_E_INVALID, std::string(name) + " shell " + std::to_string(i) + " has atom index " +
                                            std::to_string(b->shell_atom[i]) + " outside [0, natm)");
        if (b->shell_l[i] < 0)
            return fail(DFJK_E_INVALID, std::string(name) + " shell " + std::to_string(i) + " has l < 0");
        if (b->shell_l[i] > lmax)
            return fail(DFJK_E_UNSUPPORTED, std::string(name) + " shell " + std::to_string(i) + " has l = " +
                                                std::to_string(b->shell_l[i]) + " > " + std::to_string(lmax));
        const double e = b->shell_exp[i];
        if (!(e > 0.0) || !std::isfinite(e))
            return fail(DFJK_E_INVALID, std::string(name) + " shell " + std::to_string(i) +
                                            " has a non-positive or non-finite exponent");
    }
    return DFJK_OK;
}

static int create(int32_t natm, const double *coords, const dfjk_basis *ao, const dfjk_basis *aux,
                  const dfjk_options *opt, dfjk_plan **out)
{
    if (!out) return fail(DFJK_E_INVALID, "out is NULL");
    if (natm <= 0) return fail(DFJK_E_INVALID, "natm must be positive");
    if (!coords) return fail(DFJK_E_INVALID, "coords is NULL");
    for (int i = 0; i < 3 * natm; ++i)
        if (!std::isfinite(coords[i])) return fail(DFJK_E_INVALID, "coords contain a non-finite value");
    int rc = validate_basis(ao, natm, kMaxLAO, "AO");
    if (rc) return rc;
    rc = validate_basis(aux, natm, kMaxLAux, "aux");
    if (rc) return rc;
    double thresh = 1e-14;
    if (opt) {
        thresh = opt->schwarz_thresh;
        if (!(thresh >= 0.0) || !std::isfinite(thresh))
            return fail(DFJK_E_INVALID, "schwarz_thresh must be finite and >= 0");
        if (opt->aux_slab < 0) return fail(DFJK_E_INVALID, "aux_slab must be >= 0");
        if (opt->k_tile != 0 && opt->k_tile != 64 && opt->k_tile != 96 && opt->k_tile != 128)
            return fail(DFJK_E_INVALID, "k_tile must be 0, 64, 96 or 128");
    }
    int64_t nao = 0, naux = 0;
    for (int i = 0; i < ao->nshell; ++i) nao += 2 * ao->shell_l[i] + 1;
    for (int i = 0; i < aux->nshell; ++i) naux += 2 * aux->shell_l[i] + 1;
    if (nao > 32768 || naux > 65536 || (int64_t)ao->nshell * (ao->nshell + 1) / 2 > INT32_MAX / 2)
        return fail(DFJK_E_UNSUPPORTED, "basis too large for this version");

    auto *h = new dfjk_plan();
    Plan &p = h->p;
    p.natm = natm;
    p.coords.assign(coords, coords + 3 * natm);
    p.thresh = thresh;
    p.aux_slab = opt ? opt->aux_slab : 0;
    p.k_tile = opt ? opt->k_tile : 0;
    p.nsh_ao = ao->nshell;
    p.ao_atom.assign(ao->shell_atom, ao->shell_atom + ao->nshell);
    p.ao_l.assign(ao->shell_l, ao->shell_l + ao->nshell);
    p.ao_exp.assign(ao->shell_exp, ao->shell_exp + ao->nshell);
    p.ao_off.resize(ao->nshell + 1);
    p.ao_off[0] = 0;
    for (int i = 0; i < ao->nshell; ++i) p.ao_off[i + 1] = p.ao_off[i] + 2 * p.ao_l[i] + 1;
    p.nao = nao;
    p.ao_norm.resize(ao->nshell);
    p.ao_x.resize(ao->nshell); p.ao_y.resize(ao->nshell); p.ao_z.resize(ao->nshell);
    for (int i = 0; i < ao->nshell; ++i) {
        p.ao_norm[i] = shell_norm(p.ao_l[i], p.ao_exp[i]);
        p.ao_x[i] = coords[3 * p.ao_atom[i]];
        p.ao_y[i] = coords[3 * p.ao_atom[i] + 1];
        p.ao_z[i] = coords[3 * p.ao_atom[i] + 2];
    }
    // aux shells ordered by l (stable): every angular class is a contiguous range
    p.nsh_aux = aux->nshell;
    std::vector<int32_t> caller_off(aux->nshell + 1, 0);
    for (int i = 0; i < aux->nshell; ++i) caller_off[i + 1] = caller_off[i] + 2 * aux->shell_l[i] + 1;
    p.ax_caller.resize(aux->nshell);
    std::iota(p.ax_caller.begin(), p.ax_caller.end(), 0);
    std::stable_sort(p.ax_caller.begin(), p.ax_caller.end(),
                     [&](int a, int b) { return aux->shell_l[a] < aux->shell_l[b]; });
    p.ax_l.resize(aux->nshell); p.ax_exp.resize(aux->nshell); p.ax_norm.resize(aux->nshell);
    p.ax_x.resize(aux->nshell); p.ax_y.resize(aux->nshell); p.ax_z.resize(aux->nshell);
    p.ax_off.resize(aux->nshell + 1);
    p.ax_off[0] = 0;
    p.ax_fn_caller.clear();
    for (int l = 0; l <= kMaxLAux; ++l) p.ax_class[l] = {0, 0};
    for (int i = 0; i < aux->nshell; ++i) {
        const int c = p.ax_caller[i];
        p.ax_l[i] = aux->shell_l[c];
        p.ax_exp[i] = aux->shell_exp[c];
        p.ax_norm[i] = shell_norm(p.ax_l[i], p.ax_exp[i]);
        const int at = aux->shell_atom[c];
        p.ax_x[i] = coords[3 * at]; p.ax_y[i] = coords[3 * at + 1]; p.ax_z[i] = coords[3 * at + 2];
        p.ax_off[i + 1] = p.ax_off[i] + 2 * p.ax_l[i] + 1;
        for (int m = 0; m < 2 * p.ax_l[i] + 1; ++m) p.ax_fn_caller.push_back(caller_off[c] + m);
    }
    for (int l = 0; l <= kMaxLAux; ++l) {
        int b = -1, e = -1;
        for (int i = 0; i < aux->nshell; ++i)
            if (p.ax_l[i] == l) { if (b < 0) b = i; e = i + 1; }
        p.ax_class[l] = (b < 0) ? ClassRange{0, 0} : ClassRange{b, e};
    }
    p.naux = naux;
    p.naux_pad = (int64_t)align_up((size_t)naux, kPadAux);
    p.npair_all = (int64_t)ao->nshell * (ao->nshell + 1) / 2;
    p.stage = 0;
    *out = h;
    return DFJK_OK;
}

// ---------------------------------------------------------------------------
// Screening.

struct ScreenLayout {
    size_t o_ao[7], o_ax[7], o_qp, o_qa, o_dsh, bytes;
};

static ScreenLayout screen_layout(const Plan &p)
{
    ScreenLayout L{};
    size_t off = 0;
    auto take = [&](size_t b) { off = align_up(off, 256); size_t o = off; off += b; return o; };
    for (int i = 0; i < 5; ++i) L.o_ao[i] = take(p.nsh_ao * 8);     // exp x y z norm
    L.o_ao[5] = take(p.nsh_ao * 4);                                  // l
    L.o_ao[6] = take((p.nsh_ao + 1) * 4);                            // off
    for (int i = 0; i < 5; ++i) L.o_ax[i] = take(p.nsh_aux * 8);
    L.o_ax[5] = take(p.nsh_aux * 4);
    L.o_ax[6] = take((p.nsh_aux + 1) * 4);
    L.o_qp = take((size_t)p.npair_all * 8);
    L.o_qa = take((size_t)p.nsh_aux * 8);
    L.o_dsh = take((size_t)p.nsh_ao * 4 + 4);                        // d shells
    L.bytes = align_up(off, 256);
    return L;
}

// One shell pair that the screen keeps.
struct KeptPair { int a, b, cls; double q; };

// By class, then by descending q (positive), stable: a radix sort on the bits of q,
// which order as the values do.  32 waters keep 13,000 pairs: 0.53 ms by comparisons,
// 0.15 by digits; its 7 passes over 2,048 counters take 10 us, what 4 waters' 800
// pairs take by comparisons.
static void sort_kept(std::vector<KeptPair> &keep)
{
    const size_t n = keep.size();
    if (n < 1024) {
        std::stable_sort(keep.begin(), keep.end(), [](const KeptPair &u, const KeptPair &v) {
            return u.cls != v.cls ? u.cls < v.cls : u.q > v.q;
        });
        return;
    }
    std::vector<std::pair<uint64_t, uint32_t>> k(n), t(n);
    for (size_t i = 0; i < n; ++i) {
        uint64_t bits;
        std::memcpy(&bits, &keep[i].q, 8);
        k[i] = {~bits, (uint32_t)i};
    }
    constexpr int kBits = 11;
    std::vector<uint32_t> start((size_t)1 << kBits);
    for (int shift = 0; shift < 64 + kBits; shift += kBits) {
        // the last pass is by class
        const bool by_class = shift >= 64;
        auto digit = [&](const std::pair<uint64_t, uint32_t> &e) -> uint32_t {
            return by_class ? (uint32_t)keep[e.second].cls : (uint32_t)(e.first >> shift) & ((1u << kBits) - 1);
        };
        std::fill(start.begin(), start.end(), 0u);
        for (const auto &e : k) ++start[digit(e)];
        uint32_t sum = 0;
        for (auto &c : start) { const uint32_t v = c; c = sum; sum += v; }
        for (const auto &e : k) t[start[digit(e)]++] = e;
        k.swap(t);
    }
    std::vector<KeptPair> out(n);
    for (size_t i = 0; i < n; ++i) out[i] = keep[k[i].second];
    keep.swap(out);
}

static int screen(Plan &p, void *scratch, size_t bytes, hipStream_t s)
{
    int dev = 0;
    int rc = check_device(&dev);
    if (rc) return rc;
    const double *boys_dev = nullptr;
    Error er = ensure_device_constants(dev, &boys_dev);
    if (er.code) return fail(er.code, er.msg);
    const ScreenLayout L = screen_layout(p);
    if (!scratch) return fail(DFJK_E_INVALID, "screen scratch is NULL");
    p.dir.ready = false;   // direct-path tables follow the screening
    if (bytes < L.bytes) return fail(DFJK_E_OOM, "screen scratch too small: need " + std::to_string(L.bytes));
    char *b = static_cast<char *>(scratch);
    auto up = [&](size_t o, const void *src, size_t n) { return hipMemcpyAsync(b + o, src, n, hipMemcpyHostToDevice, s); };
    // the shell tables lie back to back from offset 0: packed on the host
    // into one buffer (kept until the synchronisation below), one copy
    const size_t tab_end = L.o_ax[6] + (p.nsh_aux + 1) * 4;
    std::vector<char> tab(tab_end, 0);
    auto put = [&](size_t o, const void *src, size_t n) { if (n) std::memcpy(tab.data() + o, src, n); };
    put(L.o_ao[0], p.ao_exp.data(), p.nsh_ao * 8);
    put(L.o_ao[1], p.ao_x.data(), p.nsh_ao * 8);
    put(L.o_ao[2], p.ao_y.data(), p.nsh_ao * 8);
    put(L.o_ao[3], p.ao_z.data(), p.nsh_ao * 8);
    put(L.o_ao[4], p.ao_norm.data(), p.nsh_ao * 8);
    put(L.o_ao[5], p.ao_l.data(), p.nsh_ao * 4);
    put(L.o_ao[6], p.ao_off.data(), (p.nsh_ao + 1) * 4);
    put(L.o_ax[0], p.ax_exp.data(), p.nsh_aux * 8);
    put(L.o_ax[1], p.ax_x.data(), p.nsh_aux * 8);
    put(L.o_ax[2], p.ax_y.data(), p.nsh_aux * 8);
    put(L.o_ax[3], p.ax_z.data(), p.nsh_aux * 8);
    put(L.o_ax[4], p.ax_norm.data(), p.nsh_aux * 8);
    put(L.o_ax[5], p.ax_l.data(), p.nsh_aux * 4);
    put(L.o_ax[6], p.ax_off.data(), (p.nsh_aux + 1) * 4);
    HIP_OR_FAIL(up(0, tab.data(), tab_end));
    ShellsDev ao{(double *)(b + L.o_ao[0]), (double *)(b + L.o_ao[1]), (double *)(b + L.o_ao[2]),
                 (double *)(b + L.o_ao[3]), (double *)(b + L.o_ao[4]), nullptr,
                 (int32_t *)(b + L.o_ao[5]), (int32_t *)(b + L.o_ao[6])};
    ShellsDev ax{(double *)(b + L.o_ax[0]), (double *)(b + L.o_ax[1]), (double *)(b + L.o_ax[2]),
                 (double *)(b + L.o_ax[3]), (double *)(b + L.o_ax[4]), nullptr,
                 (int32_t *)(b + L.o_ax[5]), (int32_t *)(b + L.o_ax[6])};
    double *qp = (double *)(b + L.o_qp), *qa = (double *)(b + L.o_qa);
    std::vector<int32_t> dsh;
    for (int32_t i = 0; i < p.nsh_ao; ++i)
        if (p.ao_l[i] == 2) dsh.push_back(i);
    if (!dsh.empty()) HIP_OR_FAIL(up(L.o_dsh, dsh.data(), dsh.size() * 4));
    launch_schwarz(p.npair_all, ao, (const int32_t *)(b + L.o_dsh), (int32_t)dsh.size(), p.nsh_aux, ax, qp, qa, s);
    HIP_OR_FAIL(hipGetLastError());
    p.q_pair.resize(p.npair_all);
    p.q_aux.resize(p.nsh_aux);
    HIP_OR_FAIL(hipMemcpyAsync(p.q_pair.data(), qp, p.npair_all * 8, hipMemcpyDeviceToHost, s));
    HIP_OR_FAIL(hipMemcpyAsync(p.q_aux.data(), qa, p.nsh_aux * 8, hipMemcpyDeviceToHost, s));
    HIP_OR_FAIL(hipStreamSynchronize(s));

    // ---- compaction: keep pairs whose best triplet bound reaches the threshold
    const double qmax_aux = *std::max_element(p.q_aux.begin(), p.q_aux.end());
    std::vector<KeptPair> keep;
    keep.reserve(p.npair_all / 4 + 16);
    for (int a = 0; a < p.nsh_ao; ++a)
        for (int bb = 0; bb <= a; ++bb) {
            const double q = p.q_pair[(int64_t)a * (a + 1) / 2 + bb];
            if (!(q * qmax_aux >= p.thresh)) continue;
            int x = a, y = bb;
            if (p.ao_l[x] < p.ao_l[y]) std::swap(x, y);
            const int la = p.ao_l[x], lb = p.ao_l[y];
            const int cls = la == 0 ? 0 : (la == 1 ? 1 + lb : 3 + lb);
            keep.push_back({x, y, cls, q});
        }
    sort_kept(keep);
    const size_t np = keep.size();
    p.sp_a.resize(np); p.sp_b.resize(np); p.sp_f0.resize(np); p.sp_q.resize(np);
    for (int c = 0; c < 6; ++c) p.sp_class[c] = {0, 0};
    int64_t f = 0;
    p.triplets_kept = 0;
    // kept triplets of a pair: the aux shells with q * Q_P >= thresh, a suffix of
    // the ascending Q_P (the predicate is monotone in Q_P) that shrinks as q
    // falls along a class
    std::vector<double> qa_sorted(p.q_aux);
    std::sort(qa_sorted.begin(), qa_sorted.end());
    auto first = qa_sorted.begin();
    for (size_t i = 0; i < np; ++i) {
        if (i > 0 && keep[i].cls != keep[i - 1].cls) first = qa_sorted.begin();
        p.sp_a[i] = keep[i].a; p.sp_b[i] = keep[i].b; p.sp_q[i] = keep[i].q;
        p.sp_f0[i] = (int32_t)f;
        f += (int64_t)(2 * p.ao_l[keep[i].a] + 1) * (2 * p.ao_l[keep[i].b] + 1);
        while (first != qa_sorted.end() && !(keep[i].q * *first >= p.thresh)) ++first;
        p.triplets_kept += qa_sorted.end() - first;
    }
    for (int c = 0; c < 6; ++c) {
        int bgn = -1, end = -1;
        for (size_t i = 0; i < np; ++i)
            if (keep[i].cls == c) { if (bgn < 0) bgn = (int)i; end = (int)i + 1; }
        p.sp_class[c] = bgn < 0 ? ClassRange{0, 0} : ClassRange{bgn, end};
    }
    if (f > INT32_MAX) return fail(DFJK_E_UNSUPPORTED, "too many significant function pairs");
    p.nf = f;
    p.nf_pad = (int64_t)align_up((size_t)std::max<int64_t>(f, 1), kPadF);
    // rows: AO functions and weights
    p.f_mu.assign(p.nf_pad, 0); p.f_nu.assign(p.nf_pad, 0); p.f_w.assign(p.nf_pad, 0.0);
    for (size_t i = 0; i < np; ++i) {
        const int a = p.sp_a[i], bb = p.sp_b[i];
        const int na = 2 * p.ao_l[a] + 1, nb = 2 * p.ao_l[bb] + 1;
        for (int ma = 0; ma < na; ++ma)
            for (int mb = 0; mb < nb; ++mb) {
                const int32_t row = p.sp_f0[i] + ma * nb + mb;
                p.f_mu[row] = p.ao_off[a] + ma; p.f_nu[row] = p.ao_off[bb] + mb;
                p.f_w[row] = (a == bb) ? 1.0 : 2.0;
            }
    }
    // half-transform lists: for AO function mu, every kept partner nu (both
    // orientations of a pair) with its row, by increasing nu.  Each shell's
    // kept pairs by increasing partner shell give its functions' lists in order:
    // dealt out by partner shell, so nothing is sorted.
    std::vector<int32_t> adj_off(p.nsh_ao + 1, 0);
    for (size_t i = 0; i < np; ++i) {
        ++adj_off[p.sp_a[i] + 1];
        if (p.sp_a[i] != p.sp_b[i]) ++adj_off[p.sp_b[i] + 1];
    }
    for (int x = 0; x < p.nsh_ao; ++x) adj_off[x + 1] += adj_off[x];
    using Partner = std::pair<int32_t, int32_t>;   // (partner shell, pair)
    std::vector<Partner> any(adj_off[p.nsh_ao]), adj(adj_off[p.nsh_ao]);
    {
        std::vector<int32_t> cur(adj_off.begin(), adj_off.end() - 1);
        for (size_t i = 0; i < np; ++i) {
            const int a = p.sp_a[i], bb = p.sp_b[i];
            any[cur[a]++] = {bb, (int32_t)i};
            if (a != bb) any[cur[bb]++] = {a, (int32_t)i};
        }
        cur.assign(adj_off.begin(), adj_off.end() - 1);
        for (int y = 0; y < p.nsh_ao; ++y)
            for (int32_t e = adj_off[y]; e < adj_off[y + 1]; ++e) adj[cur[any[e].first]++] = {y, any[e].second};
    }
    // every list in whole chunks for the half transform: padding entries pair a
    // real B row with the zero coefficient row nao
    p.hk_off.assign(p.nao + 1, 0);
    for (int x = 0; x < p.nsh_ao; ++x) {
        int32_t len = 0;
        for (int32_t e = adj_off[x]; e < adj_off[x + 1]; ++e) len += 2 * p.ao_l[adj[e].first] + 1;
        len = (int32_t)align_up((size_t)len, kHtChunk);
        for (int32_t mu = p.ao_off[x]; mu < p.ao_off[x + 1]; ++mu) p.hk_off[mu + 1] = p.hk_off[mu] + len;
    }
    p.hk_row.resize(p.hk_off[p.nao]);
    p.hk_nu.resize(p.hk_off[p.nao]);
    for (int x = 0; x < p.nsh_ao; ++x)
        for (int32_t mu = p.ao_off[x]; mu < p.ao_off[x + 1]; ++mu) {
            const int mx = mu - p.ao_off[x];
            int32_t at = p.hk_off[mu];
            for (int32_t e = adj_off[x]; e < adj_off[x + 1]; ++e) {
                const int y = adj[e].first, i = adj[e].second;
                const int ny = 2 * p.ao_l[y] + 1;
                const int nb = 2 * p.ao_l[p.sp_b[i]] + 1;
                const bool x_first = p.sp_a[i] == x;   // mu in the pair's first shell
                for (int my = 0; my < ny; ++my, ++at) {
                    p.hk_nu[at] = p.ao_off[y] + my;
                    p.hk_row[at] = p.sp_f0[i] + (x_first ? mx * nb + my : my * nb + mx);
                }
            }
            for (; at < p.hk_off[mu + 1]; ++at) {
                p.hk_row[at] = p.hk_row[at - 1];
                p.hk_nu[at] = (int32_t)p.nao;
            }
        }
    if (p.hk_row.empty()) { p.hk_row.push_back(0); p.hk_nu.push_back(0); }
    // half-transform workgroups run longest k list first (fewer short tails)
    p.hk_order.resize(p.nao);
    std::iota(p.hk_order.begin(), p.hk_order.end(), 0);
    std::stable_sort(p.hk_order.begin(), p.hk_order.end(), [&](int32_t a, int32_t b) {
        return p.hk_off[a + 1] - p.hk_off[a] > p.hk_off[b + 1] - p.hk_off[b];
    });
    p.device = dev;
    int ncu = 0;
    if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && ncu > 0)
        p.num_cus = ncu;
    p.stage = 1;
    return DFJK_OK;
}

// ---------------------------------------------------------------------------
// Setup.

struct SetupLayout {
    size_t o[40];
    size_t bytes;
};

// rows: function-pair rows of the U and B buffers (nf_pad: whole; fewer for
// the host-resident setup, which forms B one row block at a time into two
// B buffers and factors the metric in the buffer of L).
static SetupLayout setup_layout(const Plan &p, Plan *carve, int64_t rows = -1)
{
    const bool blocked = rows >= 0;
    if (!blocked) rows = p.nf_pad;
    SetupLayout L{};
    size_t off = 0;
    int k = 0;
    auto take = [&](size_t b) { off = align_up(off, 256); size_t o = off; off += std::max<size_t>(b, 8); L.o[k++] = o; return o; };
    const size_t na = p.nsh_ao, nx = p.nsh_aux, np = std::max<size_t>(p.sp_a.size(), 1);
    take(na * 8); take(na * 8); take(na * 8); take(na * 8); take(na * 8);   // 0-4 ao exp x y z norm
    take(na * 4); take((na + 1) * 4);                                        // 5-6 ao l off
    take(nx * 8); take(nx * 8); take(nx * 8); take(nx * 8); take(nx * 8); take(nx * 8); // 7-12 ax exp x y z norm q
    take(nx * 4); take((nx + 1) * 4);                                        // 13-14 ax l off
    take(p.naux * 4); take(p.naux * 4);                                      // 15-16 fn_caller, fn_internal
    take((size_t)p.nao * p.nao * 4);                                         // 17 fmap
    take(np * 4); take(np * 4); take(np * 4); take(np * 8);                  // 18-21 sp a b f0 q
    take(p.nf_pad * 4); take(p.nf_pad * 4); take(p.nf_pad * 8);              // 22-24 f mu nu w
    take((p.nao + 1) * 4); take(p.hk_row.size() * 4); take(p.hk_nu.size() * 4); // 25-27
    take((size_t)rows * p.naux_pad * 8);                                     // 28 U
    take((size_t)rows * p.naux_pad * 8 * (blocked ? 2 : 1));                 // 29 B
    take(blocked ? 8 : (size_t)p.naux_pad * p.naux_pad * 8);                 // 30 V
    take((size_t)p.naux_pad * p.naux_pad * 8);                               // 31 L
    take((size_t)p.naux_pad * p.naux_pad * 8);                               // 32 Linv
    take(64);                                                                // 33 status
    take((size_t)p.nao * 4);                                                 // 34 hk_order
    take((size_t)p.naux_pad * 64 * 8);                                       // 35 Dinv
    int64_t roff[7];
    pair_rec_offsets(p, roff);
    take((size_t)roff[6] * 8);                                               // 36 pair records
    L.bytes = align_up(off, 256);
    if (carve) {
        char *b = carve->ws;
        auto P = [&](int i) { return b + L.o[i]; };
        auto &d = carve->d;
        d.ao_exp = (double *)P(0); d.ao_x = (double *)P(1); d.ao_y = (double *)P(2); d.ao_z = (double *)P(3);
        d.ao_norm = (double *)P(4); d.ao_l = (int32_t *)P(5); d.ao_off = (int32_t *)P(6);
        d.ax_exp = (double *)P(7); d.ax_x = (double *)P(8); d.ax_y = (double *)P(9); d.ax_z = (double *)P(10);
        d.ax_norm = (double *)P(11); d.ax_q = (double *)P(12); d.ax_l = (int32_t *)P(13); d.ax_off = (int32_t *)P(14);
        d.ax_fn_caller = (int32_t *)P(15); d.ax_fn_internal = (int32_t *)P(16); d.fmap = (int32_t *)P(17);
        d.sp_a = (int32_t *)P(18); d.sp_b = (int32_t *)P(19); d.sp_f0 = (int32_t *)P(20); d.sp_q = (double *)P(21);
        d.f_mu = (int32_t *)P(22); d.f_nu = (int32_t *)P(23); d.f_w = (double *)P(24);
        d.hk_off = (int32_t *)P(25); d.hk_row = (int32_t *)P(26); d.hk_nu = (int32_t *)P(27);
        d.U = (double *)P(28); d.B = (double *)P(29); d.V = (double *)P(blocked ? 31 : 30); d.L = (double *)P(31);
        d.Linv = (double *)P(32); d.status = (int32_t *)P(33); d.hk_order = (int32_t *)P(34);
        d.Dinv = (double *)P(35);
        d.pair_rec = (double *)P(36);
    }
    return L;
}

// Host staging kept alive for the asynchronous uploads of one setup: the
// tables of each contiguous run of workspace slots packed into one buffer.
struct Staging {
    std::vector<int32_t> fn_internal;
    std::vector<int32_t> status;
    std::vector<char> run[3];
};

// Uploads of the host tables and the function-pair map (both setups).
static int setup_upload(Plan &p, Staging &st, hipStream_t s)
{
    st.fn_internal.assign(p.naux, 0);
    for (int64_t i = 0; i < p.naux; ++i) st.fn_internal[p.ax_fn_caller[i]] = (int32_t)i;
    st.status.assign(16, INT_MAX);
    auto &d = p.d;
    // Three runs of adjacent workspace slots (0-16: shells and function maps;
    // 18-27: pair, function-pair and partner tables; 33-34: status and the
    // partner order), each packed on the host and copied at once.  The
    // buffers live in `st` until the setup's synchronisation.
    auto pack = [&](std::vector<char> &buf, const char *first, const char *end,
                    std::initializer_list<std::tuple<const void *, const void *, size_t>> parts) {
        buf.assign((size_t)(end - first), 0);
        for (const auto &t : parts) {
            const ptrdiff_t o = (const char *)std::get<0>(t) - first;
            const size_t n = std::get<2>(t);
            if (o < 0 || (size_t)o + n > buf.size()) return hipErrorInvalidValue;   // a slot outside its run
            if (n) std::memcpy(buf.data() + o, std::get<1>(t), n);
        }
        return hipMemcpyAsync(const_cast<char *>(first), buf.data(), buf.size(), hipMemcpyHostToDevice, s);
    };
    const size_t np = p.sp_a.size();
    HIP_OR_FAIL(pack(st.run[0], (const char *)d.ao_exp, (const char *)(d.ax_fn_internal + p.naux), {
        {d.ao_exp, p.ao_exp.data(), p.nsh_ao * 8}, {d.ao_x, p.ao_x.data(), p.nsh_ao * 8},
        {d.ao_y, p.ao_y.data(), p.nsh_ao * 8}, {d.ao_z, p.ao_z.data(), p.nsh_ao * 8},
        {d.ao_norm, p.ao_norm.data(), p.nsh_ao * 8}, {d.ao_l, p.ao_l.data(), p.nsh_ao * 4},
        {d.ao_off, p.ao_off.data(), (p.nsh_ao + 1) * 4},
        {d.ax_exp, p.ax_exp.data(), p.nsh_aux * 8}, {d.ax_x, p.ax_x.data(), p.nsh_aux * 8},
        {d.ax_y, p.ax_y.data(), p.nsh_aux * 8}, {d.ax_z, p.ax_z.data(), p.nsh_aux * 8},
        {d.ax_norm, p.ax_norm.data(), p.nsh_aux * 8}, {d.ax_q, p.q_aux.data(), p.nsh_aux * 8},
        {d.ax_l, p.ax_l.data(), p.nsh_aux * 4}, {d.ax_off, p.ax_off.data(), (p.nsh_aux + 1) * 4},
        {d.ax_fn_caller, p.ax_fn_caller.data(), p.naux * 4}, {d.ax_fn_internal, st.fn_internal.data(), p.naux * 4}}));
    HIP_OR_FAIL(pack(st.run[1], (const char *)d.sp_a, (const char *)(d.hk_nu + p.hk_nu.size()), {
        {d.sp_a, p.sp_a.data(), np * 4}, {d.sp_b, p.sp_b.data(), np * 4},
        {d.sp_f0, p.sp_f0.data(), np * 4}, {d.sp_q, p.sp_q.data(), np * 8},
        {d.f_mu, p.f_mu.data(), p.nf_pad * 4}, {d.f_nu, p.f_nu.data(), p.nf_pad * 4},
        {d.f_w, p.f_w.data(), p.nf_pad * 8},
        {d.hk_off, p.hk_off.data(), (p.nao + 1) * 4}, {d.hk_row, p.hk_row.data(), p.hk_row.size() * 4},
        {d.hk_nu, p.hk_nu.data(), p.hk_nu.size() * 4}}));
    HIP_OR_FAIL(pack(st.run[2], (const char *)d.status, (const char *)(d.hk_order + p.nao), {
        {d.status, st.status.data(), 16 * 4}, {d.hk_order, p.hk_order.data(), p.nao * 4}}));
    launch_fmap(p, s);
    return DFJK_OK;
}

// The metric's Cholesky status, read after the factor (synchronises).
static int setup_status(Plan &p, Staging &st, hipStream_t s)
{
    HIP_OR_FAIL(hipGetLastError());
    HIP_OR_FAIL(hipMemcpyAsync(st.status.data(), p.d.status, 16 * 4, hipMemcpyDeviceToHost, s));
    HIP_OR_FAIL(hipStreamSynchronize(s));
    if (st.status[0] != INT_MAX) {
        const int internal = st.status[0];
        const int caller = internal < p.naux ? p.ax_fn_caller[internal] : internal;
        p.stage = 1;
        return fail(DFJK_E_NOT_POSDEF, "metric Cholesky: pivot <= 0 at aux function " + std::to_string(caller) +
                                           " (internal index " + std::to_string(internal) + ")");
    }
    return DFJK_OK;
}

// Checks of one plan's setup, before anything is enqueued.
static int setup_check(const Plan &p, const void *ws, size_t bytes, const double **boys_dev)
{
    int dev = 0;
    int rc = check_device(&dev);
    if (rc) return rc;
    if (dev != p.device) return fail(DFJK_E_STATE, "setup called on a different device than screen");
    Error er = ensure_device_constants(dev, boys_dev);
    if (er.code) return fail(er.code, er.msg);
    const SetupLayout L0 = setup_layout(p, nullptr);
    if (!ws) return fail(DFJK_E_INVALID, "workspace is NULL");
    if (bytes < L0.bytes) return fail(DFJK_E_OOM, "workspace too small: need " + std::to_string(L0.bytes));
    return DFJK_OK;
}

// The workspace carved into the plan's device tables, the host tables uploaded.
static int setup_begin(Plan &p, void *ws, size_t bytes, const double *boys_dev, Staging &st, hipStream_t s)
{
    p.ws = static_cast<char *>(ws);
    p.ws_bytes = bytes;
    setup_layout(p, &p);
    p.d.boys = boys_dev;
    return setup_upload(p, st, s);
}

// Pad rows (f >= nf) and columns of U to zero; the integrals write every
// other element (zeros for screened triplets).
static void zero_u_pads(const Plan &p, hipStream_t s)
{
    launch_zero_rect(p.d.U, p.naux_pad, 0, p.nf, p.naux, p.naux_pad, s);
    launch_zero_rect(p.d.U, p.naux_pad, p.nf, p.nf_pad, 0, p.naux_pad, s);
}

static int setup(Plan &p, void *ws, size_t bytes, hipStream_t s)
{
    const double *boys_dev = nullptr;
    int rc = setup_check(p, ws, bytes, &boys_dev);
    if (rc) return rc;
    Staging st;
    rc = setup_begin(p, ws, bytes, boys_dev, st, s);
    if (rc) return rc;
    auto &d = p.d;

    // U: zero the pad rows (f >= nf) and columns; the integrals write every
    // other element (zeros for screened triplets).  They run on the side
    // stream beside the metric and its factor (a chain of small,
    // latency-bound launches); the inverse follows them there, each block
    // row of L^{-1} as soon as its factor step is done, and the side stream
    // is joined before the whitening.  The chain is the longer of the two for a
    // small molecule, so its first steps are enqueued before the integrals' launches.
    Profiler &pr = p.prof;
    pr.stream = s;
    pr.mark(ST_SETUP, true);
    const bool side = side_stream(p);
    hipStream_t is = side ? p.j_stream : s;
    if (side) {
        HIP_OR_FAIL(hipEventRecord(p.ev_jfork, s));
        HIP_OR_FAIL(hipStreamWaitEvent(is, p.ev_jfork, 0));
    }
    auto integrals = [&] {
        pr.stream = is;
        pr.mark(ST_INT3C, true);
        zero_u_pads(p, is);
        launch_pair_records(p, is);
        launch_int3c(p, is);
        pr.mark(ST_INT3C, false);
        pr.stream = s;
    };
    if (!side) integrals();
    pr.mark(ST_METRIC, true);
    launch_metric_pad(d.V, p.naux, p.naux_pad, s);
    launch_int2c(p, s);
    HIP_OR_FAIL(hipMemcpyAsync(d.L, d.V, (size_t)p.naux_pad * p.naux_pad * 8, hipMemcpyDeviceToDevice, s));
    pr.mark(ST_METRIC, false);
    // factor steps on s, then (side stream) the same block rows of L^{-1},
    // which read only what the factor steps up to theirs wrote; handed over
    // kInvGroup steps at a time (fewer cross-stream events).  The stage of the
    // inverse is then the span of its steps, beside the factor.
    // Up to 2 kInvGroup steps (512 auxiliary functions) the inverse follows the
    // factor on s: crossing the streams costs what the overlap saves (setup of 4
    // waters 405 us against 400 to 410 with hand-overs of 2 or 3 steps, of one
    // water 210 against 235).
    constexpr int64_t kInvGroup = 4;
    const int64_t nblk = p.naux_pad / 64;
    const bool inv_on_s = !side || nblk <= 2 * kInvGroup;
    pr.mark(ST_CHOL, true);
    for (int64_t k = 0, done = 0; k < nblk; ++k) {
        cholesky_step(d.L, p.naux_pad, k, d.status, d.Dinv, s);
        if (inv_on_s || ((k + 1) % kInvGroup != 0 && k + 1 != nblk)) continue;
        if (done == 0) {
            integrals();
            trtri_begin(d.Linv, p.naux_pad, is);
        }
        HIP_OR_FAIL(hipEventRecord(p.ev_jfork, s));
        HIP_OR_FAIL(hipStreamWaitEvent(is, p.ev_jfork, 0));
        pr.stream = is;
        if (done == 0) pr.mark(ST_TRTRI, true);
        for (; done <= k; ++done) trtri_step(d.L, d.Linv, d.Dinv, p.naux_pad, done, is);
        pr.stream = s;
    }
    launch_zero_upper(d.L, p.naux_pad, s);
    pr.mark(ST_CHOL, false);
    if (inv_on_s) {
        if (side) integrals();
        pr.mark(ST_TRTRI, true);
        trtri_begin(d.Linv, p.naux_pad, s);
        for (int64_t k = 0; k < nblk; ++k) trtri_step(d.L, d.Linv, d.Dinv, p.naux_pad, k, s);
        pr.mark(ST_TRTRI, false);
    } else {
        pr.stream = is;
        pr.mark(ST_TRTRI, false);
        pr.stream = s;
    }
    if (side) {
        HIP_OR_FAIL(hipEventRecord(p.ev_jdone, is));
        HIP_OR_FAIL(hipStreamWaitEvent(s, p.ev_jdone, 0));
    }
    pr.mark(ST_WHITEN, true);
    launch_whiten(d.U, d.Linv, d.B, p.nf_pad, p.naux_pad, s);
    pr.mark(ST_WHITEN, false);
    pr.mark(ST_SETUP, false);
    rc = setup_status(p, st, s);
    if (rc) return rc;
    p.stage = 2;
    return DFJK_OK;
}

// Setup of several plans: the pair records and three-centre integrals of all
// of them in shared launches per class on `s`, then each plan's metric,
// factor, inverse and whitening on its side stream (in turn on `s` where the
// plan has none), joined back into `s`.  Every step is the one dfjk_setup
// runs, on the same elements, so each plan ends bitwise as after its own
// setup.  All checks come before anything is enqueued.
static int setup_batch(int n, Plan *const *ps, void *const *ws, const size_t *bytes, hipStream_t s)
{
    std::vector<const double *> boys(n, nullptr);
    for (int i = 0; i < n; ++i) {
        for (int j = 0; j < i; ++j)
            if (ps[j] == ps[i]) return fail(DFJK_E_INVALID, "plan " + std::to_string(i) + " given twice");
        const int rc = setup_check(*ps[i], ws[i], bytes[i], &boys[i]);
        if (rc) return fail(rc, "plan " + std::to_string(i) + ": " + g_last_error);
    }
    std::vector<Staging> st(n);
    for (int i = 0; i < n; ++i) {
        const int rc = setup_begin(*ps[i], ws[i], bytes[i], boys[i], st[i], s);
        if (rc) return rc;
        zero_u_pads(*ps[i], s);
    }
    std::vector<const Plan *> cp(ps, ps + n);
    launch_pair_records_plans(cp.data(), n, s);
    launch_int3c_plans(cp.data(), n, s);
    HIP_OR_FAIL(hipGetLastError());
    // each plan's chain of small, latency-bound launches beside the others
    std::vector<hipStream_t> cs(n, s);
    for (int i = 0; i < n; ++i) {
        Plan &p = *ps[i];
        if (!side_stream(p)) continue;
        HIP_OR_FAIL(hipEventRecord(p.ev_jfork, s));
        HIP_OR_FAIL(hipStreamWaitEvent(p.j_stream, p.ev_jfork, 0));
        cs[i] = p.j_stream;
    }
    for (int i = 0; i < n; ++i) {
        Plan &p = *ps[i];
        auto &d = p.d;
        const hipStream_t c = cs[i];
        launch_metric_pad(d.V, p.naux, p.naux_pad, c);
        launch_int2c(p, c);
        HIP_OR_FAIL(hipMemcpyAsync(d.L, d.V, (size_t)p.naux_pad * p.naux_pad * 8, hipMemcpyDeviceToDevice, c));
        launch_cholesky(d.L, p.naux_pad, d.status, d.Dinv, c);
        launch_trtri(d.L, d.Linv, d.Dinv, p.naux_pad, c);
        launch_whiten(d.U, d.Linv, d.B, p.nf_pad, p.naux_pad, c);
        if (c != s) {
            HIP_OR_FAIL(hipEventRecord(p.ev_jdone, c));
            HIP_OR_FAIL(hipStreamWaitEvent(s, p.ev_jdone, 0));
        }
    }
    int first_bad = DFJK_OK;
    std::string msg;
    for (int i = 0; i < n; ++i) {
        const int rc = setup_status(*ps[i], st[i], s);
        if (rc == DFJK_E_NOT_POSDEF) {
            if (first_bad == DFJK_OK) { first_bad = rc; msg = "plan " + std::to_string(i) + ": " + g_last_error; }
            continue;
        }
        if (rc) return rc;
        ps[i]->stage = 2;
    }
    if (first_bad) return fail(first_bad, msg);
    return DFJK_OK;
}

// ---------------------------------------------------------------------------
// Four-centre direct path: shell-pair lists and the layout of their tables.

struct DirectLists {
    std::vector<int32_t> sa[6], sb[6];
    std::vector<double> q[6];
    int64_t quartets = 0;
};

// Pairs a >= b whose largest quartet bound Q_ab max Q_cd reaches the
// threshold, per class (la >= lb orientation), by descending Q_ab; and the
// number of (bra, ket) pair combinations with Q_ab Q_cd >= threshold.
static DirectLists direct_lists(const Plan &p)
{
    DirectLists d;
    const double qmax = p.q_pair.empty() ? 0.0 : *std::max_element(p.q_pair.begin(), p.q_pair.end());
    struct Rec { int a, b; double q; };
    std::vector<Rec> rec[6];
    for (int a = 0; a < p.nsh_ao; ++a)
        for (int bb = 0; bb <= a; ++bb) {
            const double q = p.q_pair[(int64_t)a * (a + 1) / 2 + bb];
            if (!(q * qmax >= p.thresh)) continue;
            int x = a, y = bb;
            if (p.ao_l[x] < p.ao_l[y]) std::swap(x, y);
            const int la = p.ao_l[x], lb = p.ao_l[y];
            rec[la == 0 ? 0 : (la == 1 ? 1 + lb : 3 + lb)].push_back({x, y, q});
        }
    for (int c = 0; c < 6; ++c) {
        std::stable_sort(rec[c].begin(), rec[c].end(), [](const Rec &u, const Rec &v) { return u.q > v.q; });
        for (const Rec &r : rec[c]) { d.sa[c].push_back(r.a); d.sb[c].push_back(r.b); d.q[c].push_back(r.q); }
    }
    // every list is sorted descending, so the partners of one pair are a prefix
    for (int cb = 0; cb < 6; ++cb)
        for (int ck = 0; ck < 6; ++ck) {
            const std::vector<double> &qb = d.q[cb], &qk = d.q[ck];
            size_t m = qk.size();
            for (double x : qb) {
                while (m > 0 && !(x * qk[m - 1] >= p.thresh)) --m;
                d.quartets += (int64_t)m;
            }
        }
    return d;
}

static constexpr int kDirLA[6] = {0, 1, 1, 2, 2, 2}, kDirLB[6] = {0, 0, 1, 0, 1, 2};

struct DirectTables {
    size_t o_int[6][4], o_dbl[6][5], o_Eb[6], o_Ek[6];
    size_t o_sh[5], o_shoff, bytes;
    int32_t npad[6];
    int64_t herm_off[6], herm_total;
};

static DirectTables direct_tables(const Plan &p, const DirectLists &d)
{
    DirectTables T{};
    size_t off = 0;
    auto take = [&](size_t b) { off = align_up(off, 256); size_t o = off; off += b; return o; };
    T.herm_total = 0;
    for (int c = 0; c < 6; ++c) {
        const int64_t n = (int64_t)d.q[c].size();
        const int32_t npad = (int32_t)align_up((size_t)std::max<int64_t>(n, 1), 64);
        const int lab = kDirLA[c] + kDirLB[c];
        const int64_t nh = (int64_t)(lab + 1) * (lab + 2) * (lab + 3) / 6;
        const int64_t nf = (int64_t)(2 * kDirLA[c] + 1) * (2 * kDirLB[c] + 1);
        T.npad[c] = npad;
        for (int k = 0; k < 4; ++k) T.o_int[c][k] = take((size_t)npad * 4);
        for (int k = 0; k < 5; ++k) T.o_dbl[c][k] = take((size_t)npad * 8);
        T.o_Eb[c] = take((size_t)(nf * nh * npad) * 8);
        T.o_Ek[c] = take((size_t)(nf * nh * npad) * 8);
        T.herm_off[c] = T.herm_total;
        T.herm_total += nh * npad;
    }
    for (int k = 0; k < 5; ++k) T.o_sh[k] = take((size_t)std::max(p.nsh_ao, 1) * 8);
    T.o_shoff = take((size_t)(p.nsh_ao + 1) * 4);
    T.bytes = align_up(off, 256);
    return T;
}

}  // namespace dfjk

// ---------------------------------------------------------------------------
// The build that allocates nothing (dfjk_build_static).  Its scratch is this
// file-scope device array, one copy per GPU the library runs on, held until
// the process ends.  In host code the array's name is not a device address:
// the address comes from hipGetSymbolAddress, asked once per device with
// that device current, and only that address is handed to kernels.

namespace dfjk {
constexpr size_t kStaticScratchBytes = DFJK_STATIC_SCRATCH_BYTES;
}
static __device__ __align__(256) unsigned char scratch[dfjk::kStaticScratchBytes];

namespace dfjk {
static std::mutex g_static_mu;
static std::map<int, char *> g_static_ptr;   // device -> device address of `scratch` there

// The device address of `scratch` on device `dev` (current), looked up on
// the first call on that device.
static int static_scratch(int dev, char **out)
{
    std::lock_guard<std::mutex> lock(g_static_mu);
    const auto it = g_static_ptr.find(dev);
    if (it != g_static_ptr.end()) {
        *out = it->second;
        return DFJK_OK;
    }
    void *ptr = nullptr;
    HIP_OR_FAIL(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (!ptr) return fail(DFJK_E_DEVICE, "hipGetSymbolAddress returned no address for the static scratch");
    g_static_ptr[dev] = static_cast<char *>(ptr);
    *out = static_cast<char *>(ptr);
    return DFJK_OK;
}
}  // namespace dfjk

// ===========================================================================
// C ABI

using namespace dfjk;

extern "C" {

int dfjk_options_default(dfjk_options *opt)
{
    if (!opt) return fail(DFJK_E_INVALID, "opt is NULL");
    opt->schwarz_thresh = 1e-14;
    opt->aux_slab = 0;
    opt->k_tile = 0;
    return DFJK_OK;
}

int dfjk_plan_create(int32_t natm, const double *coords, const dfjk_basis *ao, const dfjk_basis *aux,
                     const dfjk_options *opt, dfjk_plan **out)
{
    try {
        return create(natm, coords, ao, aux, opt, out);
    } catch (const std::exception &e) {
        return fail(DFJK_E_INVALID, std::string("plan_create: ") + e.what());
    }
}

int dfjk_plan_info(const dfjk_plan *plan, dfjk_info *info)
{
    if (!plan || !info) return fail(DFJK_E_INVALID, "NULL argument");
    const Plan &p = plan->p;
    info->nao = p.nao;
    info->naux = p.naux;
    info->naux_pad = p.naux_pad;
    info->nshell_pairs = p.npair_all;
    info->sig_shell_pairs = (int64_t)p.sp_a.size();
    info->nf = p.nf;
    info->triplets_kept = p.triplets_kept;
    info->stage = p.stage;
    return DFJK_OK;
}

int dfjk_plan_aux_order(const dfjk_plan *plan, int32_t *out)
{
    if (!plan || !out) return fail(DFJK_E_INVALID, "NULL argument");
    for (int64_t i = 0; i < plan->p.naux; ++i) out[i] = plan->p.ax_fn_caller[i];
    return DFJK_OK;
}

int dfjk_screen_bytes(const dfjk_plan *plan, size_t *bytes)
{
    if (!plan || !bytes) return fail(DFJK_E_INVALID, "NULL argument");
    *bytes = screen_layout(plan->p).bytes;
    return DFJK_OK;
}

int dfjk_screen(dfjk_plan *plan, void *d_scratch, size_t bytes, void *stream)
{
    if (!plan) return fail(DFJK_E_INVALID, "plan is NULL");
    try {
        return screen(plan->p, d_scratch, bytes, static_cast<hipStream_t>(stream));
    } catch (const std::exception &e) {
        return fail(DFJK_E_INVALID, std::string("screen: ") + e.what());
    }
}

int dfjk_setup_bytes(const dfjk_plan *plan, size_t *bytes)
{
    if (!plan || !bytes) return fail(DFJK_E_INVALID, "NULL argument");
    if (plan->p.stage < 1) return fail(DFJK_E_STATE, "setup_bytes needs a screened plan");
    *bytes = setup_layout(plan->p, nullptr).bytes;
    return DFJK_OK;
}

// Host-resident setup: row blocks of at most `rows` function-pair rows (at
// pair boundaries; the pad rows f >= nf in the last blocks).
static std::vector<std::pair<int64_t, int32_t>> host_setup_blocks(const Plan &p, int64_t rows)
{
    // (first row, first pair) of every block, closed by (nf_pad, npairs)
    std::vector<std::pair<int64_t, int32_t>> b;
    const int32_t np = (int32_t)p.sp_a.size();
    int64_t f0 = 0;
    b.push_back({0, 0});
    for (int32_t i = 0; i < np; ++i) {
        const int64_t end = (i + 1 < np) ? p.sp_f0[i + 1] : p.nf;
        if (end - f0 > rows) {
            f0 = p.sp_f0[i];
            b.push_back({f0, i});
        }
    }
    for (int64_t f = std::max<int64_t>(p.nf, f0); f < p.nf_pad;) {   // pad rows: zeros
        if (p.nf_pad - f0 <= rows) break;
        f0 = std::max<int64_t>(f, f0 + rows);
        if (f0 >= p.nf_pad) break;
        b.push_back({f0, np});
        f = f0;
    }
    b.push_back({p.nf_pad, np});
    return b;
}

static int64_t host_setup_rows(const Plan &p, size_t max_device_bytes)
{
    if (max_device_bytes == 0) return p.nf_pad;
    const size_t fixed = setup_layout(p, nullptr, 0).bytes + 4096;
    const size_t per_row = (size_t)3 * p.naux_pad * 8;
    if (max_device_bytes <= fixed) return 0;
    return std::min<int64_t>((int64_t)((max_device_bytes - fixed) / per_row), p.nf_pad);
}

int dfjk_setup_host_bytes(const dfjk_plan *plan, size_t max_device_bytes, size_t *host_bytes, size_t *device_bytes)
{
    if (!plan || !host_bytes || !device_bytes) return fail(DFJK_E_INVALID, "NULL argument");
    const Plan &p = plan->p;
    if (p.stage < 1) return fail(DFJK_E_STATE, "setup_host_bytes needs a screened plan");
    const int64_t rows = host_setup_rows(p, max_device_bytes);
    if (rows < kMaxPairRows)
        return fail(DFJK_E_OOM, "max_device_bytes leaves room for fewer rows than one shell pair holds");
    *host_bytes = (size_t)p.nf_pad * p.naux_pad * 8;
    *device_bytes = setup_layout(p, nullptr, rows).bytes;
    return DFJK_OK;
}

int dfjk_setup_host(dfjk_plan *plan, void *h_pinned, size_t host_bytes, void *d_workspace, size_t device_bytes,
                    void *stream)
{
    if (!plan) return fail(DFJK_E_INVALID, "plan is NULL");
    Plan &p = plan->p;
    if (p.stage < 1) return fail(DFJK_E_STATE, "setup needs a screened plan (call dfjk_screen)");
    if (p.host_B) return fail(DFJK_E_STATE, "B is already host-resident");
    if (!h_pinned || !d_workspace) return fail(DFJK_E_INVALID, "NULL buffer");
    if (host_bytes < (size_t)p.nf_pad * p.naux_pad * 8) return fail(DFJK_E_OOM, "host buffer too small");
    // the widest row blocks whose workspace fits device_bytes
    int64_t rows = host_setup_rows(p, device_bytes);
    while (rows >= kMaxPairRows && setup_layout(p, nullptr, rows).bytes > device_bytes) --rows;
    if (rows < kMaxPairRows) return fail(DFJK_E_OOM, "workspace too small for one shell pair's rows");
    int dev = 0;
    int rc = check_device(&dev);
    if (rc) return rc;
    if (dev != p.device) return fail(DFJK_E_STATE, "setup called on a different device than screen");
    const double *boys_dev = nullptr;
    Error er = ensure_device_constants(dev, &boys_dev);
    if (er.code) return fail(er.code, er.msg);
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (!p.copy_stream) {
        HIP_OR_FAIL(hipStreamCreateWithFlags(&p.copy_stream, hipStreamNonBlocking));
        for (hipEvent_t *e : {&p.ev_ready[0], &p.ev_ready[1], &p.ev_free[0], &p.ev_free[1], &p.ev_start})
            HIP_OR_FAIL(hipEventCreateWithFlags(e, hipEventDisableTiming));
    }
    p.ws = static_cast<char *>(d_workspace);
    p.ws_bytes = device_bytes;
    setup_layout(p, &p, rows);
    p.d.boys = boys_dev;
    Staging st;
    rc = setup_upload(p, st, s);
    if (rc) return rc;
    auto &d = p.d;
    Profiler &pr = p.prof;
    pr.stream = s;
    // metric and its factor (V is formed in the buffer of L)
    pr.mark(ST_METRIC, true);
    launch_metric_pad(d.L, p.naux, p.naux_pad, s);
    launch_int2c(p, s);
    pr.mark(ST_METRIC, false);
    pr.mark(ST_CHOL, true);
    launch_cholesky(d.L, p.naux_pad, d.status, d.Dinv, s);
    pr.mark(ST_CHOL, false);
    pr.mark(ST_TRTRI, true);
    launch_trtri(d.L, d.Linv, d.Dinv, p.naux_pad, s);
    pr.mark(ST_TRTRI, false);
    rc = setup_status(p, st, s);
    if (rc) return rc;
    // row blocks: U rows of the block's pairs, B = U L^-T, then the block's
    // rows of every aux slab to the host (slab-major [slab][f][plen]) on the
    // copy stream, two B buffers so a block's copies overlap the next block
    int64_t slab = p.aux_slab > 0 ? (int64_t)align_up((size_t)p.aux_slab, kPadAux) : 1024;
    if (slab > p.naux_pad) slab = p.naux_pad;
    double *h = static_cast<double *>(h_pinned);
    const auto blocks = host_setup_blocks(p, rows);
    launch_pair_records(p, s);
    for (size_t bi = 0; bi + 1 < blocks.size(); ++bi) {
        const int64_t f0 = blocks[bi].first, f1 = blocks[bi + 1].first;
        const int32_t i0 = blocks[bi].second, i1 = blocks[bi + 1].second;
        const int j = (int)(bi & 1);
        double *Bj = d.B + (size_t)j * rows * p.naux_pad;
        if (bi >= 2) HIP_OR_FAIL(hipStreamWaitEvent(s, p.ev_free[j], 0));
        pr.mark(ST_INT3C, true);
        const int64_t fv = std::min<int64_t>(std::max<int64_t>(p.nf - f0, 0), f1 - f0);   // rows of real pairs
        launch_zero_rect(d.U, p.naux_pad, 0, fv, p.naux, p.naux_pad, s);
        launch_zero_rect(d.U, p.naux_pad, fv, f1 - f0, 0, p.naux_pad, s);
        if (i1 > i0) launch_int3c_rows(p, d.U, f0, i0, i1, s);
        pr.mark(ST_INT3C, false);
        pr.mark(ST_WHITEN, true);
        launch_whiten(d.U, d.Linv, Bj, f1 - f0, p.naux_pad, s);
        pr.mark(ST_WHITEN, false);
        HIP_OR_FAIL(hipEventRecord(p.ev_ready[j], s));
        HIP_OR_FAIL(hipStreamWaitEvent(p.copy_stream, p.ev_ready[j], 0));
        for (int64_t pb = 0; pb < p.naux_pad; pb += slab) {
            const int64_t plen = std::min<int64_t>(slab, p.naux_pad - pb);
            HIP_OR_FAIL(hipMemcpy2DAsync(h + (size_t)p.nf_pad * pb + (size_t)f0 * plen, plen * 8, Bj + pb,
                                         p.naux_pad * 8, plen * 8, f1 - f0, hipMemcpyDeviceToHost, p.copy_stream));
        }
        HIP_OR_FAIL(hipEventRecord(p.ev_free[j], p.copy_stream));
    }
    HIP_OR_FAIL(hipGetLastError());
    HIP_OR_FAIL(hipStreamSynchronize(p.copy_stream));
    HIP_OR_FAIL(hipStreamSynchronize(s));
    // the plan now builds as after dfjk_offload; the tables stay in the workspace
    p.d.U = p.d.B = p.d.V = p.d.L = p.d.Linv = p.d.Dinv = p.d.pair_rec = nullptr;
    p.d.fmap = nullptr;
    p.hB = h;
    p.host_slab = slab;
    p.host_B = true;
    p.stage = 2;
    return DFJK_OK;
}

int dfjk_setup(dfjk_plan *plan, void *d_workspace, size_t bytes, void *stream)
{
    if (!plan) return fail(DFJK_E_INVALID, "plan is NULL");
    if (plan->p.stage < 1) return fail(DFJK_E_STATE, "setup needs a screened plan (call dfjk_screen)");
    if (plan->p.host_B) return fail(DFJK_E_STATE, "setup after dfjk_offload is not supported");
    try {
        return setup(plan->p, d_workspace, bytes, static_cast<hipStream_t>(stream));
    } catch (const std::exception &e) {
        return fail(DFJK_E_INVALID, std::string("setup: ") + e.what());
    }
}

int dfjk_setup_batch(int32_t n, dfjk_plan *const *plans, void *const *d_workspaces, const size_t *bytes,
                     void *stream)
{
    if (n < 1 || !plans || !d_workspaces || !bytes) return fail(DFJK_E_INVALID, "n < 1 or a NULL array");
    std::vector<Plan *> ps(n);
    for (int32_t i = 0; i < n; ++i) {
        if (!plans[i]) return fail(DFJK_E_INVALID, "plan " + std::to_string(i) + " is NULL");
        if (plans[i]->p.stage < 1)
            return fail(DFJK_E_STATE, "plan " + std::to_string(i) + ": setup needs a screened plan");
        if (plans[i]->p.host_B)
            return fail(DFJK_E_STATE, "plan " + std::to_string(i) + ": setup after dfjk_offload is not supported");
        ps[i] = &plans[i]->p;
    }
    try {
        return setup_batch(n, ps.data(), d_workspaces, bytes, static_cast<hipStream_t>(stream));
    } catch (const std::exception &e) {
        return fail(DFJK_E_INVALID, std::string("setup_batch: ") + e.what());
    }
}

int dfjk_build_bytes(const dfjk_plan *plan, int32_t nocc, int32_t precision, int32_t with_density,
                     size_t *bytes)
{
    if (!plan || !bytes) return fail(DFJK_E_INVALID, "NULL argument");
    const Plan &p = plan->p;
    if (p.stage < 1) return fail(DFJK_E_STATE, "build_bytes needs a screened plan");
    if (!valid_precision(precision)) return fail(DFJK_E_INVALID, "unknown precision");
    if (with_density && precision != DFJK_FP64)
        return fail(DFJK_E_UNSUPPORTED, "the density route runs in FP64 only");
    if (with_density && p.host_B) return fail(DFJK_E_UNSUPPORTED, "the density route needs a device-resident B");
    if (!with_density && (nocc < 1 || nocc > p.nao)) return fail(DFJK_E_INVALID, "nocc must be in [1, nao]");
    *bytes = build_layout(p, nocc, precision, with_density != 0).bytes;
    return DFJK_OK;
}

int dfjk_build(dfjk_plan *plan, const double *d_C, int32_t nocc, const double *d_D, int32_t precision,
               double *d_J, double *d_K, double *d_E, void *d_scratch, size_t scratch_bytes, void *stream)
{
    if (!plan) return fail(DFJK_E_INVALID, "plan is NULL");
    Plan &p = plan->p;
    if (p.stage < 2) return fail(DFJK_E_STATE, "build needs a set-up plan (call dfjk_setup)");
    if ((d_C == nullptr) == (d_D == nullptr)) return fail(DFJK_E_INVALID, "give exactly one of C and D");
    if (!d_J || !d_K || !d_E) return fail(DFJK_E_INVALID, "an output pointer is NULL");
    if (!d_scratch) return fail(DFJK_E_INVALID, "scratch is NULL");
    if (!valid_precision(precision)) return fail(DFJK_E_INVALID, "unknown precision");
    const bool withD = d_D != nullptr;
    if (withD && precision != DFJK_FP64) return fail(DFJK_E_UNSUPPORTED, "the density route runs in FP64 only");
    if (!withD && (nocc < 1 || nocc > p.nao)) return fail(DFJK_E_INVALID, "nocc must be in [1, nao]");
    int dev = 0;
    int rc = check_device(&dev);
    if (rc) return rc;
    if (dev != p.device) return fail(DFJK_E_STATE, "build called on a different device than setup");
    if (withD && p.host_B) return fail(DFJK_E_UNSUPPORTED, "the density route needs a device-resident B");
    const BuildLayout L = build_layout(p, nocc, precision, withD);
    if (scratch_bytes < L.bytes) return fail(DFJK_E_OOM, "scratch too small: need " + std::to_string(L.bytes));
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (p.host_B) launch_build_hostB(p, L, d_C, d_J, d_K, d_E, static_cast<char *>(d_scratch), s);
    else launch_build(p, L, d_C, d_D, d_J, d_K, d_E, static_cast<char *>(d_scratch), s);
    HIP_OR_FAIL(hipGetLastError());
    return DFJK_OK;
}

// Scratch of dfjk_build_checked: the larger of the int8 and FP64 build
// layouts (the FP64 redo reuses the region), then the bound's work.
static size_t checked_layouts(const Plan &p, int32_t nocc, BuildLayout &L8, BuildLayout &L64)
{
    L8 = build_layout(p, nocc, DFJK_MIXED_INT8, false);
    L64 = build_layout(p, nocc, DFJK_FP64, false);
    const size_t base = align_up(std::max(L8.bytes, L64.bytes), 256);
    L8.norms = true;
    L8.o_norms = base;
    return base + align_up(i8_bound_work_doubles(p.nao, nocc) * 8, 256);
}

int dfjk_build_checked_bytes(const dfjk_plan *plan, int32_t nocc, size_t *bytes)
{
    if (!plan || !bytes) return fail(DFJK_E_INVALID, "NULL argument");
    const Plan &p = plan->p;
    if (p.stage < 1) return fail(DFJK_E_STATE, "build_checked_bytes needs a screened plan");
    if (nocc < 1 || nocc > p.nao) return fail(DFJK_E_INVALID, "nocc must be in [1, nao]");
    BuildLayout L8, L64;
    *bytes = checked_layouts(p, nocc, L8, L64);
    return DFJK_OK;
}

int dfjk_build_checked(dfjk_plan *plan, const double *d_C, int32_t nocc, double budget, double *d_J, double *d_K,
                       double *d_E, void *d_scratch, size_t scratch_bytes, void *stream, int32_t *chosen,
                       double *bound)
{
    if (!plan) return fail(DFJK_E_INVALID, "plan is NULL");
    Plan &p = plan->p;
    if (p.stage < 2) return fail(DFJK_E_STATE, "build needs a set-up plan (call dfjk_setup)");
    if (!d_C || !d_J || !d_K || !d_E || !d_scratch || !chosen || !bound)
        return fail(DFJK_E_INVALID, "a pointer argument is NULL");
    if (nocc < 1 || nocc > p.nao) return fail(DFJK_E_INVALID, "nocc must be in [1, nao]");
    if (!(budget > 0.0)) return fail(DFJK_E_INVALID, "budget must be > 0");
    int dev = 0;
    int rc = check_device(&dev);
    if (rc) return rc;
    if (dev != p.device) return fail(DFJK_E_STATE, "build called on a different device than setup");
    BuildLayout L8, L64;
    const size_t need = checked_layouts(p, nocc, L8, L64);
    if (scratch_bytes < need) return fail(DFJK_E_OOM, "scratch too small: need " + std::to_string(need));
    hipStream_t s = static_cast<hipStream_t>(stream);
    char *scr = static_cast<char *>(d_scratch);
    double *acc = reinterpret_cast<double *>(scr + L8.o_norms);
    double *work = acc + (size_t)p.nao * (kI8Slices + 1);
    double *out = work + gram_work_doubles(nocc) + 2;
    launch_zero(acc, p.nao * (kI8Slices + 1), s);
    if (p.host_B) launch_build_hostB(p, L8, d_C, d_J, d_K, d_E, scr, s);
    else launch_build(p, L8, d_C, nullptr, d_J, d_K, d_E, scr, s);
    // FP64 sums per element: the block folds of one split, the split and
    // slab partials, and the reduction's final scaling
    const int nsums = (int)((L8.kdim / L8.nsplit_k) / kI8Block + 8 + L8.nsplit_k * L8.nslab + 4);
    launch_i8_bound(d_C, p.nao, nocc, acc, d_E, nsums, work, out, s);
    double h = 0.0;
    HIP_OR_FAIL(hipMemcpyAsync(&h, out, sizeof(double), hipMemcpyDeviceToHost, s));
    HIP_OR_FAIL(hipStreamSynchronize(s));
    *bound = h;
    if (h <= budget) {
        *chosen = DFJK_MIXED_INT8;
    } else {
        *chosen = DFJK_FP64;
        if (p.host_B) launch_build_hostB(p, L64, d_C, d_J, d_K, d_E, scr, s);
        else launch_build(p, L64, d_C, nullptr, d_J, d_K, d_E, scr, s);
    }
    HIP_OR_FAIL(hipGetLastError());
    return DFJK_OK;
}

int dfjk_build_static(dfjk_plan *plan, const double *d_C, int32_t nocc, const double *d_D, int32_t precision,
                      double *d_J, double *d_K, double *d_E, void *stream)
{
    if (!plan) return fail(DFJK_E_INVALID, "plan is NULL");
    Plan &p = plan->p;
    if (p.stage < 2) return fail(DFJK_E_STATE, "build needs a set-up plan (call dfjk_setup)");
    if ((d_C == nullptr) == (d_D == nullptr)) return fail(DFJK_E_INVALID, "give exactly one of C and D");
    if (!d_J || !d_K || !d_E) return fail(DFJK_E_INVALID, "an output pointer is NULL");
    if (!valid_precision(precision)) return fail(DFJK_E_INVALID, "unknown precision");
    const bool withD = d_D != nullptr;
    if (withD && precision != DFJK_FP64) return fail(DFJK_E_UNSUPPORTED, "the density route runs in FP64 only");
    if (!withD && (nocc < 1 || nocc > p.nao)) return fail(DFJK_E_INVALID, "nocc must be in [1, nao]");
    int dev = 0;
    int rc = check_device(&dev);
    if (rc) return rc;
    if (dev != p.device) return fail(DFJK_E_STATE, "build called on a different device than setup");
    if (withD && p.host_B) return fail(DFJK_E_UNSUPPORTED, "the density route needs a device-resident B");
    BuildLayout L{};
    if (!static_layout(p, nocc, precision, withD, L))
        return fail(DFJK_E_OOM, "dfjk_build_static: this build needs " + std::to_string(L.bytes) +
                                    " bytes of scratch even with the narrowest aux slab; the static scratch holds " +
                                    std::to_string(kStaticScratchBytes) + " (use dfjk_build with a workspace)");
    char *ws = nullptr;
    rc = static_scratch(dev, &ws);
    if (rc) return rc;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (p.host_B) launch_build_hostB(p, L, d_C, d_J, d_K, d_E, ws, s);
    else launch_build(p, L, d_C, d_D, d_J, d_K, d_E, ws, s);
    HIP_OR_FAIL(hipGetLastError());
    return DFJK_OK;
}

int dfjk_build_delta_bytes(const dfjk_plan *plan, int32_t nocc, int32_t precision, size_t *bytes)
{
    if (!plan || !bytes) return fail(DFJK_E_INVALID, "NULL argument");
    const Plan &p = plan->p;
    if (p.stage < 1) return fail(DFJK_E_STATE, "build_delta_bytes needs a screened plan");
    if (!valid_precision(precision)) return fail(DFJK_E_INVALID, "unknown precision");
    if (nocc < 1 || nocc > p.nao) return fail(DFJK_E_INVALID, "nocc must be in [1, nao]");
    *bytes = build_layout(p, nocc, precision, false, true).bytes;
    return DFJK_OK;
}

int dfjk_build_delta(dfjk_plan *plan, const double *d_C, const double *d_C0, int32_t nocc, const double *d_K0,
                     int32_t precision, double *d_J, double *d_K, double *d_E, void *d_scratch,
                     size_t scratch_bytes, void *stream)
{
    if (!plan) return fail(DFJK_E_INVALID, "plan is NULL");
    Plan &p = plan->p;
    if (p.stage < 2) return fail(DFJK_E_STATE, "build_delta needs a set-up plan (call dfjk_setup)");
    if (p.host_B) return fail(DFJK_E_UNSUPPORTED, "build_delta needs a device-resident B");
    if (!d_C || !d_C0 || !d_K0) return fail(DFJK_E_INVALID, "C, C0 and K0 are required");
    if (!d_J || !d_K || !d_E) return fail(DFJK_E_INVALID, "an output pointer is NULL");
    if (d_K == d_K0) return fail(DFJK_E_INVALID, "K must not alias K0");
    if (!d_scratch) return fail(DFJK_E_INVALID, "scratch is NULL");
    if (!valid_precision(precision)) return fail(DFJK_E_INVALID, "unknown precision");
    if (nocc < 1 || nocc > p.nao) return fail(DFJK_E_INVALID, "nocc must be in [1, nao]");
    int dev = 0;
    int rc = check_device(&dev);
    if (rc) return rc;
    if (dev != p.device) return fail(DFJK_E_STATE, "build_delta called on a different device than setup");
    BuildLayout L = build_layout(p, nocc, precision, false, true);
    if (scratch_bytes < L.bytes) return fail(DFJK_E_OOM, "scratch too small: need " + std::to_string(L.bytes));
    L.C0 = d_C0;
    L.K0 = d_K0;
    launch_build(p, L, d_C, nullptr, d_J, d_K, d_E, static_cast<char *>(d_scratch), static_cast<hipStream_t>(stream));
    HIP_OR_FAIL(hipGetLastError());
    return DFJK_OK;
}

static int check_uks(const Plan &p, int32_t na, int32_t nb, int32_t precision)
{
    if (!valid_precision(precision)) return fail(DFJK_E_INVALID, "unknown precision");
    if (na < 0 || nb < 0 || na > p.nao || nb > p.nao || na + nb == 0)
        return fail(DFJK_E_INVALID, "nocc_a, nocc_b must be in [0, nao], not both 0");
    return DFJK_OK;
}

int dfjk_build_uks_bytes(const dfjk_plan *plan, int32_t nocc_a, int32_t nocc_b, int32_t precision, size_t *bytes)
{
    if (!plan || !bytes) return fail(DFJK_E_INVALID, "NULL argument");
    const Plan &p = plan->p;
    if (p.stage < 1) return fail(DFJK_E_STATE, "build_uks_bytes needs a screened plan");
    const int rc = check_uks(p, nocc_a, nocc_b, precision);
    if (rc) return rc;
    *bytes = build_layout_uks(p, nocc_a, nocc_b, precision).bytes;
    return DFJK_OK;
}

int dfjk_build_uks(dfjk_plan *plan, const double *d_Ca, int32_t nocc_a, const double *d_Cb, int32_t nocc_b,
                   int32_t precision, double *d_J, double *d_Ka, double *d_Kb, double *d_E, void *d_scratch,
                   size_t scratch_bytes, void *stream)
{
    if (!plan) return fail(DFJK_E_INVALID, "plan is NULL");
    Plan &p = plan->p;
    if (p.stage < 2) return fail(DFJK_E_STATE, "build_uks needs a set-up plan (call dfjk_setup)");
    if (p.host_B) return fail(DFJK_E_UNSUPPORTED, "build_uks needs a device-resident B");
    int rc = check_uks(p, nocc_a, nocc_b, precision);
    if (rc) return rc;
    if ((nocc_a > 0 && !d_Ca) || (nocc_b > 0 && !d_Cb)) return fail(DFJK_E_INVALID, "C of an occupied spin is NULL");
    if (!d_J || !d_Ka || !d_Kb || !d_E) return fail(DFJK_E_INVALID, "an output pointer is NULL");
    if (d_Ka == d_Kb) return fail(DFJK_E_INVALID, "K_a and K_b must not alias");
    if (!d_scratch) return fail(DFJK_E_INVALID, "scratch is NULL");
    int dev = 0;
    rc = check_device(&dev);
    if (rc) return rc;
    if (dev != p.device) return fail(DFJK_E_STATE, "build_uks called on a different device than setup");
    const BuildLayout L = build_layout_uks(p, nocc_a, nocc_b, precision);
    if (scratch_bytes < L.bytes) return fail(DFJK_E_OOM, "scratch too small: need " + std::to_string(L.bytes));
    launch_build_uks(p, L, d_Ca, d_Cb, d_J, d_Ka, d_Kb, d_E, static_cast<char *>(d_scratch),
                     static_cast<hipStream_t>(stream));
    HIP_OR_FAIL(hipGetLastError());
    return DFJK_OK;
}

int dfjk_direct_bytes(const dfjk_plan *plan, size_t *table_bytes)
{
    if (!plan || !table_bytes) return fail(DFJK_E_INVALID, "NULL argument");
    const Plan &p = plan->p;
    if (p.stage < 1) return fail(DFJK_E_STATE, "direct_bytes needs a screened plan (call dfjk_screen)");
    *table_bytes = direct_tables(p, direct_lists(p)).bytes;
    return DFJK_OK;
}

int dfjk_direct_setup(dfjk_plan *plan, void *d_tables, size_t bytes, void *stream)
{
    if (!plan) return fail(DFJK_E_INVALID, "plan is NULL");
    Plan &p = plan->p;
    if (p.stage < 1) return fail(DFJK_E_STATE, "direct_setup needs a screened plan (call dfjk_screen)");
    if (!d_tables) return fail(DFJK_E_INVALID, "tables pointer is NULL");
    int dev = 0;
    int rc = check_device(&dev);
    if (rc) return rc;
    if (dev != p.device) return fail(DFJK_E_STATE, "direct_setup called on a different device than screen");
    const double *boys_dev = nullptr;
    Error er = ensure_device_constants(dev, &boys_dev);
    if (er.code) return fail(er.code, er.msg);
    DirectLists d = direct_lists(p);
    const DirectTables T = direct_tables(p, d);
    if (bytes < T.bytes) return fail(DFJK_E_OOM, "direct tables too small: need " + std::to_string(T.bytes));
    p.dir = DirectState{};
    hipStream_t s = static_cast<hipStream_t>(stream);
    char *b = static_cast<char *>(d_tables);
    // host staging (kept alive until the stream is synchronised below)
    std::vector<std::vector<int32_t>> ints;
    std::vector<std::vector<double>> dbls;
    for (int c = 0; c < 6; ++c) {
        const int32_t n = (int32_t)d.q[c].size(), npad = T.npad[c];
        std::vector<int32_t> offa(npad, 0), offb(npad, 0), sha(npad, 0), shb(npad, 0);
        std::vector<double> q(npad, 0.0);
        for (int32_t i = 0; i < n; ++i) {
            sha[i] = d.sa[c][i]; shb[i] = d.sb[c][i];
            offa[i] = p.ao_off[sha[i]]; offb[i] = p.ao_off[shb[i]];
            q[i] = d.q[c][i];
        }
        ints.push_back(std::move(offa)); ints.push_back(std::move(offb));
        ints.push_back(std::move(sha)); ints.push_back(std::move(shb));
        dbls.push_back(std::move(q));
        for (int k = 0; k < 4; ++k)
            HIP_OR_FAIL(hipMemcpyAsync(b + T.o_int[c][k], ints[ints.size() - 4 + k].data(), (size_t)npad * 4,
                                       hipMemcpyHostToDevice, s));
        HIP_OR_FAIL(hipMemcpyAsync(b + T.o_dbl[c][0], dbls.back().data(), (size_t)npad * 8, hipMemcpyHostToDevice, s));
        DirectClassDev &cd = p.dir.cls[c];
        cd.n = n; cd.npad = npad;
        cd.off_a = (const int32_t *)(b + T.o_int[c][0]); cd.off_b = (const int32_t *)(b + T.o_int[c][1]);
        cd.sh_a = (const int32_t *)(b + T.o_int[c][2]); cd.sh_b = (const int32_t *)(b + T.o_int[c][3]);
        cd.q = (const double *)(b + T.o_dbl[c][0]);
        cd.px = (const double *)(b + T.o_dbl[c][1]); cd.py = (const double *)(b + T.o_dbl[c][2]);
        cd.pz = (const double *)(b + T.o_dbl[c][3]); cd.p = (const double *)(b + T.o_dbl[c][4]);
        cd.Eb = (const double *)(b + T.o_Eb[c]); cd.Ek = (const double *)(b + T.o_Ek[c]);
        cd.herm_off = T.herm_off[c];
    }
    const double *sh_src[5] = {p.ao_exp.data(), p.ao_x.data(), p.ao_y.data(), p.ao_z.data(), p.ao_norm.data()};
    for (int k = 0; k < 5; ++k)
        HIP_OR_FAIL(hipMemcpyAsync(b + T.o_sh[k], sh_src[k], (size_t)p.nsh_ao * 8, hipMemcpyHostToDevice, s));
    HIP_OR_FAIL(hipMemcpyAsync(b + T.o_shoff, p.ao_off.data(), (size_t)(p.nsh_ao + 1) * 4, hipMemcpyHostToDevice, s));
    const ShellsDev ao{(const double *)(b + T.o_sh[0]), (const double *)(b + T.o_sh[1]),
                       (const double *)(b + T.o_sh[2]), (const double *)(b + T.o_sh[3]),
                       (const double *)(b + T.o_sh[4]), nullptr, nullptr, nullptr};
    launch_direct_pairs(p.dir.cls, ao, s);
    HIP_OR_FAIL(hipGetLastError());
    HIP_OR_FAIL(hipStreamSynchronize(s));
    for (int c = 0; c < 6; ++c) { p.dir.sa[c] = std::move(d.sa[c]); p.dir.sb[c] = std::move(d.sb[c]); p.dir.q[c] = std::move(d.q[c]); }
    p.dir.herm_total = T.herm_total;
    p.dir.quartets = d.quartets;
    p.dir.table_bytes = T.bytes;
    p.dir.tables = b;
    p.dir.shell_off = (const int32_t *)(b + T.o_shoff);
    p.dir.boys = boys_dev;
    p.dir.device = dev;
    p.dir.ready = true;
    return DFJK_OK;
}

int dfjk_direct_stats(const dfjk_plan *plan, int64_t *pairs, int64_t *quartets)
{
    if (!plan || !pairs || !quartets) return fail(DFJK_E_INVALID, "NULL argument");
    const Plan &p = plan->p;
    if (!p.dir.ready) return fail(DFJK_E_STATE, "direct_stats needs dfjk_direct_setup");
    for (int c = 0; c < 6; ++c) pairs[c] = p.dir.cls[c].n;
    *quartets = p.dir.quartets;
    return DFJK_OK;
}

int dfjk_direct_build_bytes(const dfjk_plan *plan, int32_t with_density, size_t *bytes)
{
    if (!plan || !bytes) return fail(DFJK_E_INVALID, "NULL argument");
    const Plan &p = plan->p;
    if (!p.dir.ready) return fail(DFJK_E_STATE, "direct_build_bytes needs dfjk_direct_setup");
    *bytes = direct_layout(p, with_density != 0).bytes;
    return DFJK_OK;
}

int dfjk_direct_build(dfjk_plan *plan, const double *d_C, int32_t nocc, const double *d_D, double *d_J,
                      double *d_K, double *d_E, void *d_scratch, size_t scratch_bytes, void *stream)
{
    if (!plan) return fail(DFJK_E_INVALID, "plan is NULL");
    Plan &p = plan->p;
    if (!p.dir.ready) return fail(DFJK_E_STATE, "direct_build needs dfjk_direct_setup");
    if ((d_C == nullptr) == (d_D == nullptr)) return fail(DFJK_E_INVALID, "give exactly one of C and D");
    if (!d_J || !d_K || !d_E) return fail(DFJK_E_INVALID, "an output pointer is NULL");
    if (d_J == d_K) return fail(DFJK_E_INVALID, "J and K must not alias");
    if (!d_scratch) return fail(DFJK_E_INVALID, "scratch is NULL");
    const bool withD = d_D != nullptr;
    if (!withD && (nocc < 1 || nocc > p.nao)) return fail(DFJK_E_INVALID, "nocc must be in [1, nao]");
    int dev = 0;
    int rc = check_device(&dev);
    if (rc) return rc;
    if (dev != p.dir.device) return fail(DFJK_E_STATE, "direct_build called on a different device than direct_setup");
    const DirectLayout L = direct_layout(p, withD);
    if (scratch_bytes < L.bytes) return fail(DFJK_E_OOM, "scratch too small: need " + std::to_string(L.bytes));
    launch_direct_build(p, L, d_C, nocc, d_D, nullptr, nullptr, nullptr, d_J, d_K, d_E, static_cast<char *>(d_scratch),
                        static_cast<hipStream_t>(stream));
    HIP_OR_FAIL(hipGetLastError());
    return DFJK_OK;
}

int dfjk_direct_build_delta_bytes(const dfjk_plan *plan, size_t *bytes)
{
    if (!plan || !bytes) return fail(DFJK_E_INVALID, "NULL argument");
    const Plan &p = plan->p;
    if (!p.dir.ready) return fail(DFJK_E_STATE, "direct_build_delta_bytes needs dfjk_direct_setup");
    *bytes = direct_layout(p, true, true).bytes;
    return DFJK_OK;
}

int dfjk_direct_build_delta(dfjk_plan *plan, const double *d_D, const double *d_D0, const double *d_J0,
                            const double *d_K0, double *d_J, double *d_K, double *d_E, void *d_scratch,
                            size_t scratch_bytes, void *stream)
{
    if (!plan) return fail(DFJK_E_INVALID, "plan is NULL");
    Plan &p = plan->p;
    if (!p.dir.ready) return fail(DFJK_E_STATE, "direct_build_delta needs dfjk_direct_setup");
    if (!d_D || !d_D0 || !d_J0 || !d_K0) return fail(DFJK_E_INVALID, "an input pointer is NULL");
    if (!d_J || !d_K || !d_E) return fail(DFJK_E_INVALID, "an output pointer is NULL");
    if (d_J == d_K) return fail(DFJK_E_INVALID, "J and K must not alias");
    if (d_J == d_J0 || d_J == d_K0 || d_K == d_J0 || d_K == d_K0)
        return fail(DFJK_E_INVALID, "the outputs must not alias J0 or K0");
    if (!d_scratch) return fail(DFJK_E_INVALID, "scratch is NULL");
    int dev = 0;
    int rc = check_device(&dev);
    if (rc) return rc;
    if (dev != p.dir.device) return fail(DFJK_E_STATE, "direct_build_delta called on a different device than direct_setup");
    const DirectLayout L = direct_layout(p, true, true);
    if (scratch_bytes < L.bytes) return fail(DFJK_E_OOM, "scratch too small: need " + std::to_string(L.bytes));
    launch_direct_build(p, L, nullptr, 0, d_D, d_D0, d_J0, d_K0, d_J, d_K, d_E, static_cast<char *>(d_scratch),
                        static_cast<hipStream_t>(stream));
    HIP_OR_FAIL(hipGetLastError());
    return DFJK_OK;
}

// Layouts of a batch: one scratch region per molecule, 256-byte aligned, in order.
static int batch_layouts(int32_t n, dfjk_plan *const *plans, const int32_t *nocc, int32_t precision, int min_stage,
                         std::vector<BuildLayout> &Ls, std::vector<size_t> &off, size_t &total)
{
    if (n < 1) return fail(DFJK_E_INVALID, "batch needs n >= 1");
    if (!plans || !nocc) return fail(DFJK_E_INVALID, "NULL argument");
    if (!valid_precision(precision)) return fail(DFJK_E_INVALID, "unknown precision");
    std::vector<const Plan *> ps(n);
    for (int i = 0; i < n; ++i) {
        if (!plans[i]) return fail(DFJK_E_INVALID, "plan " + std::to_string(i) + " is NULL");
        ps[i] = &plans[i]->p;
        if (ps[i]->stage < min_stage)
            return fail(DFJK_E_STATE, "plan " + std::to_string(i) + (min_stage > 1 ? " is not set up" : " is not screened"));
        if (ps[i]->host_B)
            return fail(DFJK_E_UNSUPPORTED, "plan " + std::to_string(i) + " has a host-resident B");
        if (nocc[i] < 1 || nocc[i] > ps[i]->nao)
            return fail(DFJK_E_INVALID, "nocc[" + std::to_string(i) + "] must be in [1, nao]");
    }
    Ls.resize(n);
    std::vector<int> ns(n, 0);
    if (precision == DFJK_FP64) {
        for (int i = 0; i < n; ++i) Ls[i] = build_layout(*ps[i], nocc[i], precision, false, false, -1, false, 0, 0);
        batch_nsplits(ps.data(), n, Ls.data(), ns.data());
    }
    off.resize(n);
    total = 0;
    for (int i = 0; i < n; ++i) {
        Ls[i] = build_layout(*ps[i], nocc[i], precision, false, false, ns[i], false, 0, 0);   // each molecule's own tile
        off[i] = align_up(total, 256);
        total = off[i] + Ls[i].bytes;
    }
    return DFJK_OK;
}

int dfjk_build_batch_bytes(int32_t n, dfjk_plan *const *plans, const int32_t *nocc, int32_t precision,
                           size_t *bytes)
{
    if (!bytes) return fail(DFJK_E_INVALID, "NULL argument");
    std::vector<BuildLayout> Ls;
    std::vector<size_t> off;
    size_t total = 0;
    const int rc = batch_layouts(n, plans, nocc, precision, 1, Ls, off, total);
    if (rc) return rc;
    *bytes = total;
    return DFJK_OK;
}

int dfjk_build_batch(int32_t n, dfjk_plan *const *plans, const double *const *d_C, const int32_t *nocc,
                     int32_t precision, double *const *d_J, double *const *d_K, double *const *d_E, void *d_scratch,
                     size_t scratch_bytes, void *stream)
{
    std::vector<BuildLayout> Ls;
    std::vector<size_t> off;
    size_t total = 0;
    int rc = batch_layouts(n, plans, nocc, precision, 2, Ls, off, total);
    if (rc) return rc;
    if (!d_C || !d_J || !d_K || !d_E) return fail(DFJK_E_INVALID, "NULL pointer array");
    for (int i = 0; i < n; ++i)
        if (!d_C[i] || !d_J[i] || !d_K[i] || !d_E[i])
            return fail(DFJK_E_INVALID, "NULL input or output of molecule " + std::to_string(i));
    if (!d_scratch) return fail(DFJK_E_INVALID, "scratch is NULL");
    if (scratch_bytes < total) return fail(DFJK_E_OOM, "scratch too small: need " + std::to_string(total));
    int dev = 0;
    rc = check_device(&dev);
    if (rc) return rc;
    std::vector<Plan *> ps(n);
    std::vector<char *> sc(n);
    for (int i = 0; i < n; ++i) {
        ps[i] = &plans[i]->p;
        if (ps[i]->device != dev) return fail(DFJK_E_STATE, "plan " + std::to_string(i) + " lives on another device");
        sc[i] = static_cast<char *>(d_scratch) + off[i];
    }
    launch_build_batch(n, ps.data(), Ls.data(), d_C, d_J, d_K, d_E, sc.data(), static_cast<hipStream_t>(stream));
    HIP_OR_FAIL(hipGetLastError());
    return DFJK_OK;
}

static size_t offload_tables_bytes(const Plan &p)
{
    size_t off = 0;
    auto take = [&](size_t b) { off = align_up(off, 256) + std::max<size_t>(b, 8); };
    take(p.nf_pad * 4); take(p.nf_pad * 4); take(p.nf_pad * 8);
    take((p.nao + 1) * 4); take(p.hk_row.size() * 4); take(p.hk_nu.size() * 4); take(p.nao * 4);
    return align_up(off, 256);
}

int dfjk_offload_bytes(const dfjk_plan *plan, size_t *host_bytes, size_t *device_bytes)
{
    if (!plan || !host_bytes || !device_bytes) return fail(DFJK_E_INVALID, "NULL argument");
    const Plan &p = plan->p;
    if (p.stage < 1) return fail(DFJK_E_STATE, "offload_bytes needs a screened plan");
    *host_bytes = (size_t)p.nf_pad * p.naux_pad * 8;
    *device_bytes = offload_tables_bytes(p);
    return DFJK_OK;
}

int dfjk_offload(dfjk_plan *plan, void *h_pinned, size_t host_bytes, void *d_tables, size_t device_bytes,
                 void *stream)
{
    if (!plan) return fail(DFJK_E_INVALID, "plan is NULL");
    Plan &p = plan->p;
    if (p.stage < 2) return fail(DFJK_E_STATE, "offload needs a set-up plan (call dfjk_setup)");
    if (p.host_B) return fail(DFJK_E_STATE, "B is already host-resident");
    if (!h_pinned || !d_tables) return fail(DFJK_E_INVALID, "NULL buffer");
    if (host_bytes < (size_t)p.nf_pad * p.naux_pad * 8) return fail(DFJK_E_OOM, "host buffer too small");
    if (device_bytes < offload_tables_bytes(p)) return fail(DFJK_E_OOM, "table buffer too small");
    int dev = 0;
    int rc = check_device(&dev);
    if (rc) return rc;
    if (dev != p.device) return fail(DFJK_E_STATE, "offload called on a different device than setup");
    hipStream_t s = static_cast<hipStream_t>(stream);
    int64_t slab = p.aux_slab > 0 ? (int64_t)align_up((size_t)p.aux_slab, kPadAux) : 1024;
    if (slab > p.naux_pad) slab = p.naux_pad;
    double *h = static_cast<double *>(h_pinned);
    for (int64_t pb = 0; pb < p.naux_pad; pb += slab) {   // slab-major: [slab][f][plen]
        const int64_t plen = std::min<int64_t>(slab, p.naux_pad - pb);
        HIP_OR_FAIL(hipMemcpy2DAsync(h + (size_t)p.nf_pad * pb, plen * 8, p.d.B + pb, p.naux_pad * 8, plen * 8,
                                     p.nf_pad, hipMemcpyDeviceToHost, s));
    }
    char *t = static_cast<char *>(d_tables);
    size_t off = 0;
    auto move = [&](auto *&ptr, size_t bytes) {
        off = align_up(off, 256);
        using T = std::remove_pointer_t<std::remove_reference_t<decltype(ptr)>>;
        T *dst = reinterpret_cast<T *>(t + off);
        const hipError_t e = hipMemcpyAsync(dst, ptr, bytes, hipMemcpyDeviceToDevice, s);
        ptr = dst;
        off += std::max<size_t>(bytes, 8);
        return e;
    };
    HIP_OR_FAIL(move(p.d.f_mu, p.nf_pad * 4));
    HIP_OR_FAIL(move(p.d.f_nu, p.nf_pad * 4));
    HIP_OR_FAIL(move(p.d.f_w, p.nf_pad * 8));
    HIP_OR_FAIL(move(p.d.hk_off, (p.nao + 1) * 4));
    HIP_OR_FAIL(move(p.d.hk_row, p.hk_row.size() * 4));
    HIP_OR_FAIL(move(p.d.hk_nu, p.hk_nu.size() * 4));
    HIP_OR_FAIL(move(p.d.hk_order, p.nao * 4));
    HIP_OR_FAIL(hipStreamSynchronize(s));
    if (!p.copy_stream) {
        HIP_OR_FAIL(hipStreamCreateWithFlags(&p.copy_stream, hipStreamNonBlocking));
        for (hipEvent_t *e : {&p.ev_ready[0], &p.ev_ready[1], &p.ev_free[0], &p.ev_free[1], &p.ev_start})
            HIP_OR_FAIL(hipEventCreateWithFlags(e, hipEventDisableTiming));
    }
    // the setup workspace is no longer referenced
    p.d.U = p.d.B = p.d.V = p.d.L = p.d.Linv = p.d.Dinv = p.d.pair_rec = nullptr;
    p.d.fmap = nullptr;
    p.ws = nullptr;
    p.ws_bytes = 0;
    p.hB = h;
    p.host_slab = slab;
    p.host_B = true;
    return DFJK_OK;
}

int dfjk_autotune_bytes(const dfjk_plan *plan, int32_t nocc, int32_t precision, size_t *bytes)
{
    if (!plan || !bytes) return fail(DFJK_E_INVALID, "NULL argument");
    const Plan &p = plan->p;
    if (p.stage < 1) return fail(DFJK_E_STATE, "autotune_bytes needs a screened plan");
    if (!valid_precision(precision)) return fail(DFJK_E_INVALID, "unknown precision");
    if (nocc < 1 || nocc > p.nao) return fail(DFJK_E_INVALID, "nocc must be in [1, nao]");
    size_t most = 0;
    for (const KShape &c : autotune_candidates(p, nocc, precision))
        most = std::max(most, build_layout(p, nocc, precision, false, false, c.nsplit, true, 0, c.tile).bytes);
    *bytes = align_up(most, 256) + (size_t)2 * p.nao * p.nao * 8 + 256;   // + J, K and E of the trial builds
    return DFJK_OK;
}

int dfjk_build_shape(const dfjk_plan *plan, int32_t nocc, int32_t precision, int32_t *shape)
{
    if (!plan || !shape) return fail(DFJK_E_INVALID, "NULL argument");
    const Plan &p = plan->p;
    if (p.stage < 1) return fail(DFJK_E_STATE, "build_shape needs a screened plan");
    if (!valid_precision(precision)) return fail(DFJK_E_INVALID, "unknown precision");
    if (nocc < 1 || nocc > p.nao) return fail(DFJK_E_INVALID, "nocc must be in [1, nao]");
    const BuildLayout L = build_layout(p, nocc, precision, false);
    shape[0] = L.ktile;
    shape[1] = L.nsplit_k;
    shape[2] = (int32_t)L.slab;
    shape[3] = (int32_t)L.nslab;
    return DFJK_OK;
}

int dfjk_autotune(dfjk_plan *plan, const double *d_C, int32_t nocc, int32_t precision, void *d_scratch,
                  size_t scratch_bytes, void *stream, int32_t *chosen, int32_t *ncand, int32_t *cand, double *ms)
{
    if (!plan || !d_C || !d_scratch) return fail(DFJK_E_INVALID, "NULL argument");
    Plan &p = plan->p;
    if (p.stage < 2) return fail(DFJK_E_STATE, "autotune needs a set-up plan (call dfjk_setup)");
    size_t need = 0;
    int rc = dfjk_autotune_bytes(plan, nocc, precision, &need);
    if (rc) return rc;
    if (scratch_bytes < need) return fail(DFJK_E_OOM, "scratch too small: need " + std::to_string(need));
    int dev = 0;
    rc = check_device(&dev);
    if (rc) return rc;
    if (dev != p.device) return fail(DFJK_E_STATE, "autotune called on a different device than setup");
    hipStream_t s = static_cast<hipStream_t>(stream);
    const std::vector<KShape> cands = autotune_candidates(p, nocc, precision);
    size_t most = 0;
    for (const KShape &c : cands)
        most = std::max(most, build_layout(p, nocc, precision, false, false, c.nsplit, true, 0, c.tile).bytes);
    char *scr = static_cast<char *>(d_scratch);
    double *J = reinterpret_cast<double *>(scr + align_up(most, 256));
    double *K = J + (size_t)p.nao * p.nao;
    double *E = K + (size_t)p.nao * p.nao;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    HIP_OR_FAIL(hipEventCreate(&e0));
    HIP_OR_FAIL(hipEventCreate(&e1));
    const bool prof = p.prof.on;
    p.prof.on = false;
    std::vector<double> t(cands.size(), 0.0);
    hipError_t err = hipSuccess;
    for (size_t i = 0; i < cands.size() && err == hipSuccess; ++i) {
        const BuildLayout L = build_layout(p, nocc, precision, false, false, cands[i].nsplit, true, 0, cands[i].tile);
        const int reps = 3;
        for (int r = 0; r <= reps; ++r) {            // the first build warms up
            if (r == 1) err = hipEventRecord(e0, s);
            if (p.host_B) launch_build_hostB(p, L, d_C, J, K, E, scr, s);
            else launch_build(p, L, d_C, nullptr, J, K, E, scr, s);
        }
        if (err == hipSuccess) err = hipEventRecord(e1, s);
        if (err == hipSuccess) err = hipEventSynchronize(e1);
        float m = 0.f;
        if (err == hipSuccess) err = hipEventElapsedTime(&m, e0, e1);
        t[i] = m / reps;
    }
    p.prof.on = prof;
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    HIP_OR_FAIL(err);
    HIP_OR_FAIL(hipGetLastError());
    const size_t best = (size_t)(std::min_element(t.begin(), t.end()) - t.begin());
    p.tuned[(int64_t)nocc * 8 + precision] = cands[best];
    const auto code = [](const KShape &k) { return (int32_t)(1000 * k.tile + k.nsplit); };
    if (chosen) *chosen = code(cands[best]);
    if (ncand) {
        const int nmax = *ncand;
        *ncand = (int32_t)cands.size();
        for (int i = 0; i < (int)cands.size() && i < nmax; ++i) {
            if (cand) cand[i] = code(cands[i]);
            if (ms) ms[i] = t[i];
        }
    }
    return DFJK_OK;
}

int dfjk_export(const dfjk_plan *plan, int32_t kind, double *d_out, void *stream)
{
    if (!plan || !d_out) return fail(DFJK_E_INVALID, "NULL argument");
    if (plan->p.stage < 2) return fail(DFJK_E_STATE, "export needs a set-up plan");
    if (plan->p.host_B) return fail(DFJK_E_STATE, "the tensors were moved to the host (dfjk_offload)");
    if (kind < DFJK_EXPORT_INT3C || kind > DFJK_EXPORT_CHOL) return fail(DFJK_E_INVALID, "unknown export kind");
    launch_export(plan->p, kind, d_out, static_cast<hipStream_t>(stream));
    HIP_OR_FAIL(hipGetLastError());
    return DFJK_OK;
}

int dfjk_sample(const dfjk_plan *plan, int32_t kind, int64_t n, const int32_t *d_idx, double *d_out,
                void *stream)
{
    if (!plan || !d_idx || !d_out) return fail(DFJK_E_INVALID, "NULL argument");
    if (plan->p.stage < 2) return fail(DFJK_E_STATE, "sample needs a set-up plan");
    if (plan->p.host_B) return fail(DFJK_E_STATE, "the tensors were moved to the host (dfjk_offload)");
    if (kind != DFJK_EXPORT_INT3C && kind != DFJK_EXPORT_B) return fail(DFJK_E_INVALID, "kind must be 0 or 1");
    if (n < 0) return fail(DFJK_E_INVALID, "n < 0");
    if (n == 0) return DFJK_OK;
    launch_sample(plan->p, kind, n, d_idx, d_out, static_cast<hipStream_t>(stream));
    HIP_OR_FAIL(hipGetLastError());
    return DFJK_OK;
}

int dfjk_boys(int32_t mmax, int64_t n, const double *d_T, double *d_F, void *stream)
{
    if (mmax < 0 || mmax > kBoysMMaxPublic) return fail(DFJK_E_INVALID, "mmax must be in [0, 16]");
    if (n < 0) return fail(DFJK_E_INVALID, "n < 0");
    if (n > 0 && (!d_T || !d_F)) return fail(DFJK_E_INVALID, "NULL argument");
    int dev = 0;
    int rc = check_device(&dev);
    if (rc) return rc;
    const double *tab = nullptr;
    Error er = ensure_device_constants(dev, &tab);
    if (er.code) return fail(er.code, er.msg);
    if (n == 0) return DFJK_OK;
    launch_boys_eval(mmax, n, d_T, d_F, tab, static_cast<hipStream_t>(stream));
    HIP_OR_FAIL(hipGetLastError());
    return DFJK_OK;
}

int dfjk_profile(dfjk_plan *plan, int32_t on)
{
    if (!plan) return fail(DFJK_E_INVALID, "plan is NULL");
    Profiler &pr = plan->p.prof;
    pr.on = on != 0;
    pr.rec_stage.clear();
    for (int &o : pr.open) o = -1;
    return DFJK_OK;
}

int dfjk_profile_read(dfjk_plan *plan, double *ms, int32_t *count)
{
    if (!plan || !ms || !count) return fail(DFJK_E_INVALID, "NULL argument");
    Profiler &pr = plan->p.prof;
    for (int i = 0; i < ST_COUNT; ++i) { ms[i] = 0.0; count[i] = 0; }
    for (size_t i = 0; i < pr.rec_stage.size(); ++i) {
        if (pr.open[pr.rec_stage[i]] == (int)i) continue;   // still open (a build in flight): no end yet
        HIP_OR_FAIL(hipEventSynchronize(pr.pool[2 * i + 1]));
        float t = 0.f;
        HIP_OR_FAIL(hipEventElapsedTime(&t, pr.pool[2 * i], pr.pool[2 * i + 1]));
        ms[pr.rec_stage[i]] += t;
        count[pr.rec_stage[i]] += 1;
    }
    pr.rec_stage.clear();
    for (int &o : pr.open) o = -1;
    return DFJK_OK;
}

const char *dfjk_stage_name(int32_t stage)
{
    return (stage >= 0 && stage < ST_COUNT) ? kStageNames[stage] : "";
}

int dfjk_plan_destroy(dfjk_plan *plan)
{
    if (plan) {
        for (hipEvent_t e : plan->p.prof.pool) (void)hipEventDestroy(e);
        Plan &p = plan->p;
        if (p.copy_stream) (void)hipStreamSynchronize(p.copy_stream);
        if (p.ht_stream) (void)hipStreamSynchronize(p.ht_stream);
        if (p.j_stream) (void)hipStreamSynchronize(p.j_stream);
        for (hipEvent_t e : {p.ev_ready[0], p.ev_ready[1], p.ev_free[0], p.ev_free[1], p.ev_start, p.ev_fork,
                             p.ev_ht[0], p.ev_ht[1], p.ev_kdone[0], p.ev_kdone[1], p.ev_jfork, p.ev_jdone})
            if (e) (void)hipEventDestroy(e);
        for (const auto &e : p.side_events) {
            (void)hipEventDestroy(e.first);
            (void)hipEventDestroy(e.second);
        }
        if (p.copy_stream) (void)hipStreamDestroy(p.copy_stream);
        if (p.ht_stream) (void)hipStreamDestroy(p.ht_stream);
        if (p.j_stream) (void)hipStreamDestroy(p.j_stream);
    }
    delete plan;
    return DFJK_OK;
}

const char *dfjk_last_error(void) { return g_last_error.c_str(); }

// Owns what dfjk_build_host allocates; everything is released on every return.
namespace {
struct HostCallState {
    dfjk_plan *plan = nullptr;
    std::vector<void *> dev;
    hipStream_t stream = nullptr;
    ~HostCallState()
    {
        if (stream) (void)hipStreamSynchronize(stream);
        for (void *q : dev) (void)hipFree(q);
        if (stream) (void)hipStreamDestroy(stream);
        dfjk_plan_destroy(plan);
    }
    hipError_t alloc(void **q, size_t n)
    {
        *q = nullptr;
        const hipError_t e = hipMalloc(q, n > 0 ? n : 1);
        if (e == hipSuccess) dev.push_back(*q);
        return e;
    }
};
}  // namespace

int dfjk_build_host(int32_t natm, const double *coords, const dfjk_basis *ao, const dfjk_basis *aux,
                    const dfjk_options *opt, const double *C, int32_t nocc, const double *D, int32_t precision,
                    double *J, double *K, double *E)
{
    if ((C == nullptr) == (D == nullptr)) return fail(DFJK_E_INVALID, "give exactly one of C and D");
    if (!J || !K || !E) return fail(DFJK_E_INVALID, "an output pointer is NULL");
    HostCallState st;
    int rc = dfjk_plan_create(natm, coords, ao, aux, opt, &st.plan);
    if (rc) return rc;
    int dev = 0;
    rc = check_device(&dev);
    if (rc) return rc;
    HIP_OR_FAIL(hipStreamCreateWithFlags(&st.stream, hipStreamNonBlocking));
    const int64_t nao = st.plan->p.nao;
    size_t n = 0;
    void *scr = nullptr, *ws = nullptr, *bscr = nullptr, *dC = nullptr, *dJ = nullptr, *dK = nullptr,
         *dE = nullptr;
    if ((rc = dfjk_screen_bytes(st.plan, &n))) return rc;
    HIP_OR_FAIL(st.alloc(&scr, n));
    if ((rc = dfjk_screen(st.plan, scr, n, st.stream))) return rc;
    if ((rc = dfjk_setup_bytes(st.plan, &n))) return rc;
    HIP_OR_FAIL(st.alloc(&ws, n));
    if ((rc = dfjk_setup(st.plan, ws, n, st.stream))) return rc;
    const bool withD = D != nullptr;
    if ((rc = dfjk_build_bytes(st.plan, nocc, precision, withD, &n))) return rc;
    HIP_OR_FAIL(st.alloc(&bscr, n));
    const size_t in_bytes = withD ? (size_t)nao * nao * 8 : (size_t)nao * nocc * 8;
    HIP_OR_FAIL(st.alloc(&dC, in_bytes));
    HIP_OR_FAIL(st.alloc(&dJ, (size_t)nao * nao * 8));
    HIP_OR_FAIL(st.alloc(&dK, (size_t)nao * nao * 8));
    HIP_OR_FAIL(st.alloc(&dE, 16));
    HIP_OR_FAIL(hipMemcpyAsync(dC, withD ? D : C, in_bytes, hipMemcpyHostToDevice, st.stream));
    rc = dfjk_build(st.plan, withD ? nullptr : static_cast<const double *>(dC), nocc,
                    withD ? static_cast<const double *>(dC) : nullptr, precision, static_cast<double *>(dJ),
                    static_cast<double *>(dK), static_cast<double *>(dE), bscr, n, st.stream);
    if (rc) return rc;
    HIP_OR_FAIL(hipMemcpyAsync(J, dJ, (size_t)nao * nao * 8, hipMemcpyDeviceToHost, st.stream));
    HIP_OR_FAIL(hipMemcpyAsync(K, dK, (size_t)nao * nao * 8, hipMemcpyDeviceToHost, st.stream));
    HIP_OR_FAIL(hipMemcpyAsync(E, dE, 16, hipMemcpyDeviceToHost, st.stream));
    HIP_OR_FAIL(hipStreamSynchronize(st.stream));
    return DFJK_OK;
}

}  // extern "C"
