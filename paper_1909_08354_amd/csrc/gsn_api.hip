// gsn_api.hip -- host side of the C ABI declared in include/gsn.h.
//
// Owns argument validation, the layout of the caller's workspace, the FP64
// tables (twiddles, per-axis |k|^2 and kinetic factors, all generated on the
// host with double cos/sin), the per-step pass schedule and its launches.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <fstream>
#include <map>
#include <mutex>
#include <new>
#include <sstream>
#include <string>
#include <vector>

#include "gsn_host.hpp"
#include "gsn_corrector_internal.hpp"

thread_local std::string g_last_error;

extern "C" const char *gsn_last_error(void) { return g_last_error.c_str(); }

template <int N, int V> static NKernels make_kernels()
{
    using C = Cfg<N, V>;
    constexpr int E = C::E, LL = C::LM_LINES, EL = C::EM_LINES;
    NKernels k;
    k.E = E;
    k.TPL = C::TPL;
    k.lm_lines = LL;
    k.em_lines = EL;
    for (int m = 0; m < 4; ++m) k.lmp[m] = k.lmp2[m] = nullptr;
    k.em_pipe = C::PIPE;
    if constexpr (V == kSmallVariant) {
        small_kernels<N, float2>(k);
        return k;
    } else {
        k.em_fwd = k_em_fft<N, E, EL, -1>;
        k.em_inv = k_em_fft<N, E, EL, 1>;
        k.density = k_density<N, E, EL, false>;
        k.density_store = k_density<N, E, EL, true>;
        k.density_real = k_density_real<N, E, EL>;
        k.phase = k_phase<N, E, EL, false, false>;
        k.phase_real = k_phase<N, E, EL, false, true>;
        k.phase_energy = k_phase<N, E, EL, true, false>;
        k.potential = k_potential<N, E, EL>;
        k.lm_fwd = k_lm<N, E, LL, LM_FWD>;
        k.lm_inv = k_lm<N, E, LL, LM_INV>;
        k.lm_kin = k_lm<N, E, LL, LM_KIN>;
        k.lm_kern = k_lm<N, E, LL, LM_KERN>;
        k.lm_kin_energy = k_lm<N, E, LL, LM_KIN_ENERGY>;
    }
    if constexpr (C::PIPE) {
        k.density = k_densityp<N, E, EL, false>;
        k.density_store = k_densityp<N, E, EL, true>;
        k.phase = k_phasep<N, E, EL, false>;
        k.phase_real = k_phasep<N, E, EL, true>;
        using T = TwoButterfly<N>;
        constexpr bool TWO = V == 3 && T::ON;
        if constexpr (TWO) {
            k.lmp2[LM_FWD] = k_lmp2<N, T::LINES, LM_FWD>;
            k.lmp2[LM_INV] = k_lmp2<N, T::LINES, LM_INV>;
            k.lmp2[LM_KIN] = k_lmp2<N, T::LINES, LM_KIN>;
            k.lmp2[LM_KERN] = k_lmp2<N, T::LINES, LM_KERN>;
            k.lmp2_lines = T::LINES;
            k.lmp2_threads = T::THREADS;
            k.lmp2_min_tiles = T::MIN_TILES;
        }
        // where the two-butterfly form has the same tiles and takes any number of
        // them, no pass is left for the one-butterfly form
        if constexpr (!(TWO && T::LINES == LL && T::MIN_TILES == 0)) {
            k.lmp[LM_FWD] = k_lmp<N, E, LL, LM_FWD, float2>;
            k.lmp[LM_INV] = k_lmp<N, E, LL, LM_INV, float2>;
            k.lmp[LM_KIN] = k_lmp<N, E, LL, LM_KIN, float2>;
            k.lmp[LM_KERN] = k_lmp<N, E, LL, LM_KERN, float2>;
        }
    }
    return k;
}

template <int N> static const NKernels *variant_table(int v)
{
    static const NKernels k[kNumVariants] = {make_kernels<N, 0>(), make_kernels<N, 1>(), make_kernels<N, 2>(),
                                             make_kernels<N, 3>(), make_kernels<N, 4>(),
                                             make_kernels<N, kSmallVariant>()};
    return &k[v];
}

const NKernels *kernels_for(int N, int v)
{
    if (v < 0 || v >= kNumVariants) v = 0;
    switch (N) {
    case 8: return variant_table<8>(v);
    case 16: return variant_table<16>(v);
    case 32: return variant_table<32>(v);
    case 64: return variant_table<64>(v);
    case 128: return variant_table<128>(v);
    case 256: return variant_table<256>(v);
    case 512: return variant_table<512>(v);
    case 1024: return variant_table<1024>(v);
    case 2048: return variant_table<2048>(v);
    default: return nullptr;
    }
}


// ------------------------------------------------------------------ passes
// After the ten passes of the model: three that carry sqrt(rho) to
// lap(sqrt rho) for the Bohm potential of Eq. (15), three that carry rho to
// lap(rho) and the x pass that forms the source gamma rho + beta lap(rho) of the
// position-dependent coupling; each runs only while its term is on (a 2-D
// grid uses only the Laplacian column passes).
enum PassId {
    P_ENTRY = 0, P_KIN_Y, P_KINETIC, P_DENSITY, P_Y_FWD_RHO, P_KERNEL,
    P_Y_INV_PHI, P_PHASE, P_EXIT, P_Y_FWD_SQRT, P_LAPLACIAN, P_Y_INV_LAP, P_Y_FWD_SRC,
    P_LAP_RHO, P_Y_INV_SRC, P_SOURCE, P_COUNT
};
static const char *kPassNames[P_COUNT] = {
    "x_entry_fft", "kinetic_y", "kinetic", "x_density", "y_fwd_rho",
    "kernel", "y_inv_phi", "x_phase", "x_exit_ifft", "y_fwd_sqrt", "laplacian", "y_inv_lap",
    "y_fwd_src", "lap_rho", "y_inv_src", "x_source"};

struct Launch {
    const void *fn;
    dim3 grid, block;
    bool em;
    EmArgs ea;
    LmArgs la;
    int pass;
};

struct StepLists {
    std::vector<Launch> entry, kin_half, kin_full, nonlin, exit_;
};

struct gsn_grid_ {
    int storage;               // GSN_C64 or GSN_C128 (FP64 storage)
    size_t esz;                // bytes per complex value in HBM (8 or 16)
    int ndim;
    int n[3];
    double L[3];
    long long P;
    int Nx, Ny, Nz;   // Nz = 1 in 2-D
    hipStream_t stream;
    int device;
    // workspace carve-up
    float2 *psi, *scratch, *half, *nyq;
    float2 *half2, *nyq2;      // sqrt(rho) -> lap(sqrt rho) spectrum (Bohm term)
    double *mass_parts, *epart;
    DevState *st;
    double2 *tw[3];            // twiddles for x, y, z lengths
    double *k2[3];             // |k_d|^2 tables
    double2 *kinF[3], *kinH[3];
    double *k2_unit;
    double2 *kin_unit;
    double2 *sct;              // sin / cos table of the pipelined phase pass
    int var[P_COUNT];          // schedule variant per pass
    int store_psi;             // 1: density pass stores real-space psi for the phase pass
    int max_density_blocks;    // over all variants (sizes the partial arrays)
    // parameters
    double a, g, dz;
    gsn_kernel kern;
    double mY2;                // squared screening mass of K; -C of Eq. (2) (may be < 0)
    double lp_cp, lp_n, lp_cb, lp_floor;   // local terms of Eq. (15)
    bool local_on, bohm_on;
    // position-dependent coupling: caller-owned device fields (null: absent)
    const float *fld_gamma, *fld_beta, *fld_V;
    bool have_dz, have_psi;
    // launch schedules
    std::vector<Launch> entry, kin_half, kin_full, nonlin, exit_, energy_rho, energy_kin;
    std::vector<Launch> pot;      // potential readout (phi pointer set per call)
    std::vector<Launch> pot_spec; // the same from x-spectral psi, ending a coarse step (see gsn_step_corrected)
    StepLists coarse;             // one coarse step of coarse_ratio * dz
    int coarse_ratio;             // 0 = no coarse schedule
    double2 *kinFc[3], *kinHc[3]; // kinetic tables of the coarse step
    DevState *st_save[2];         // device copies of the state for audits
    std::vector<char> tab;        // host copy of the workspace's tables
    char *tab_dev;
    HostObs *obs_dev, *obs_host;  // where read-outs land: workspace, or pinned host memory (may be null)
    int density_blocks;
    bool static_ws;               // workspace = the library's static array (gsn_create_static)
};


struct Layout {
    size_t psi, scratch, half, nyq, half2, nyq2, mass_parts, epart, st, obs, tables, total;
    int density_blocks, em_blocks, lm_blocks_max;
};

static gsn_status validate_shape(int ndim, const int32_t n[])
{
    if (ndim != 2 && ndim != 3) return fail(GSN_EUNSUPPORTED, "ndim must be 2 or 3");
    if (!n) return fail(GSN_EINVAL, "n is NULL");
    for (int d = 0; d < ndim; ++d)
        if (!is_pow2(n[d]) || n[d] < 8 || n[d] > 2048)
            return fail(GSN_EUNSUPPORTED,
                        "every extent must be a power of two in [8, 2048], got " + std::to_string(n[d]));
    return GSN_OK;
}

static int lm_tiles_main(int nlines, int lines_per_tile, int nouter)
{
    return ((nlines + lines_per_tile - 1) / lines_per_tile) * nouter;
}

static Layout compute_layout(int ndim, const int32_t n[], size_t esz = 8)
{
    Layout L{};
    const int Nx = n[ndim - 1], Ny = n[ndim - 2], Nz = ndim == 3 ? n[0] : 1;
    const long long P = (long long)Nx * Ny * Nz;
    const long long rows = P / Nx;
    // partial arrays are sized for the largest grid over all schedule variants
    int lmb = 0;
    for (int v = 0; v < kNumVariants; ++v) {
        const NKernels *kx = kernels_for(Nx, v), *kl = kernels_for(ndim == 3 ? Nz : Ny, v);
        const int db = (int)((rows / 2 + kx->em_lines - 1) / kx->em_lines) * kx->em_parts;
        if (db > L.density_blocks) L.density_blocks = db;
        const int eb = (int)((rows + kx->em_lines - 1) / kx->em_lines);
        if (eb > L.em_blocks) L.em_blocks = eb;
        // kinetic-energy pass over the last axis
        const int t = ndim == 3 ? lm_tiles_main(Nx, kl->lm_lines, Ny) : lm_tiles_main(Nx, kl->lm_lines, 1);
        if (t > lmb) lmb = t;
    }
    L.lm_blocks_max = lmb;
    size_t off = 0;
    L.psi = off; off = align256(off + esz * P);
    L.scratch = off; off = align256(off + esz * P);
    L.half = off; off = align256(off + esz * (P / 2));
    L.nyq = off; off = align256(off + esz * rows);
    L.half2 = off; off = align256(off + esz * (P / 2));
    L.nyq2 = off; off = align256(off + esz * rows);
    L.mass_parts = off; off = align256(off + 8ull * (size_t)(L.density_blocks > 1024 ? L.density_blocks : 1024));
    size_t ep = 4ull * (size_t)L.density_blocks + (size_t)lmb + 1024;
    L.epart = off; off = align256(off + 8ull * ep);
    L.st = off; off = align256(off + sizeof(DevState));
    L.obs = off; off = align256(off + sizeof(HostObs));
    L.tables = off;
    size_t tb = 0;
    for (int d = 0; d < ndim; ++d) tb += align256(16ull * n[d]) * 5 + align256(8ull * n[d]);
    tb += 512 + 512 + 16 * kSinCosTable;
    off = align256(off + tb);
    L.total = off;
    return L;
}

extern "C" gsn_status gsn_workspace_bytes(int ndim, const int32_t n[], size_t *bytes)
{
    gsn_status s = validate_shape(ndim, n);
    if (s) return s;
    if (!bytes) return fail(GSN_EINVAL, "bytes is NULL");
    *bytes = compute_layout(ndim, n).total;
    return GSN_OK;
}

static size_t storage_bytes(int storage) { return storage == GSN_C128 ? 16 : 8; }

extern "C" gsn_status gsn_workspace_bytes_ex(int ndim, const int32_t n[], int storage, size_t *bytes)
{
    gsn_status s = validate_shape(ndim, n);
    if (s) return s;
    if (!bytes) return fail(GSN_EINVAL, "bytes is NULL");
    if (storage != GSN_C64 && storage != GSN_C128) return fail(GSN_EINVAL, "storage must be GSN_C64 or GSN_C128");
    *bytes = compute_layout(ndim, n, storage_bytes(storage)).total;
    return GSN_OK;
}

// ------------------------------------------------------------------ schedule construction
static Seg seg_empty()
{
    Seg s;
    std::memset(&s, 0, sizeof(s));
    return s;
}

static Seg make_seg(float2 *ptr, long long es, long long ls, long long os, int nlines, int nouter,
                    int lines_per_tile)
{
    Seg s = seg_empty();
    s.ptr = ptr;
    s.es = es;
    s.ls = ls;
    s.os = os;
    s.nlines = nlines;
    s.ngroups = (nlines + lines_per_tile - 1) / lines_per_tile;
    s.ntiles = s.ngroups * nouter;
    return s;
}

static LmArgs lm_base(gsn_grid g, const double2 *tw, double scale)
{
    LmArgs a;
    std::memset(&a, 0, sizeof(a));
    a.tw = tw;
    a.scale = scale;
    a.kin1 = a.kin2 = a.kinp = g->kin_unit;
    a.k2_1 = a.k2_2 = a.k2_p = g->k2_unit;
    a.st = g->st;
    return a;
}

// The coefficients of K(k), with the scale of everything from rho to phi: 1/P for
// the transforms and 1/2 for the split of two real rows' spectra, which is stored
// without it (all powers of two, so no bit of phi depends on where they are
// applied; the passes in between have two multiplications a point less each).
static void set_kernel_args(gsn_grid g, LmArgs &a)
{
    const double s = 0.5 / (double)g->P;
    a.cN = g->kern.c_newton * s;
    a.cY = g->kern.c_yukawa * s;
    a.mY2 = g->mY2;
    a.c0 = g->kern.c_contact * s;
}

// The pipelined LM form addresses a tile with 32-bit offsets: every offset
// inside a tile, ((LINES - 1) ls + (N - 1) es) * 8 bytes, must stay below 2^31.
static bool lm_fits(const Seg &s, int N, int lines)
{
    if (s.ntiles == 0) return true;
    const long long span = ((long long)(lines - 1) * s.ls + (long long)(N - 1) * s.es) * 8 + 8;
    return span > 0 && span < (1LL << 31);
}

// Resident blocks per CU times CUs (persistent grid size); 0 if unknown.
int persistent_blocks(const void *fn, int threads)
{
    static std::mutex mu;
    static std::map<std::pair<const void *, int>, int> cache;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    std::lock_guard<std::mutex> lock(mu);
    const auto key = std::make_pair(fn, dev);
    auto it = cache.find(key);
    if (it != cache.end()) return it->second;
    int per_cu = 0, cus = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, threads, 0) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    const int n = per_cu > 0 && cus > 0 ? per_cu * cus : 0;
    cache[key] = n;
    return n;
}

// The same lines in tiles of `lines`.
static void regroup(Seg &s, int lines)
{
    if (s.ntiles == 0) return;
    const int nouter = s.ntiles / s.ngroups;
    s.ngroups = (s.nlines + lines - 1) / lines;
    s.ntiles = s.ngroups * nouter;
}

static Launch lm_launch(void (*fn)(LmArgs), const NKernels *k, LmArgs a, int pass)
{
    Launch L;
    std::memset(&L, 0, sizeof(L));
    int mode = -1;
    if (fn == k->lm_fwd) mode = LM_FWD;
    else if (fn == k->lm_inv) mode = LM_INV;
    else if (fn == k->lm_kin) mode = LM_KIN;
    else if (fn == k->lm_kern) mode = LM_KERN;
    const int N = k->E * k->TPL;
    int threads = k->lm_threads();
    bool pipe = false;
    if (mode >= 0 && k->lmp2[mode] && lm_fits(a.s0, N, k->lmp2_lines) && lm_fits(a.s1, N, k->lmp2_lines)) {
        Seg s0 = a.s0, s1 = a.s1;
        regroup(s0, k->lmp2_lines);
        regroup(s1, k->lmp2_lines);
        if (s0.ntiles + s1.ntiles >= k->lmp2_min_tiles) {
            a.s0 = s0;
            a.s1 = s1;
            fn = k->lmp2[mode];
            threads = k->lmp2_threads;
            pipe = true;
        }
    }
    if (!pipe && mode >= 0 && k->lmp[mode] && lm_fits(a.s0, N, k->lm_lines) && lm_fits(a.s1, N, k->lm_lines)) {
        fn = k->lmp[mode];
        pipe = true;
    }
    int grid = a.s0.ntiles + a.s1.ntiles;
    if (pipe) {
        const int pb = persistent_blocks((const void *)fn, threads);
        if (pb > 0 && pb < grid) grid = pb;
    }
    if (k->mass_block && a.reduce) ++grid;
    L.fn = (const void *)fn;
    L.grid = dim3(grid);
    L.block = dim3(threads);
    L.em = false;
    L.la = a;
    L.pass = pass;
    return L;
}

static Launch em_launch(void (*fn)(EmArgs), const NKernels *k, const EmArgs &a, int pass)
{
    Launch L;
    std::memset(&L, 0, sizeof(L));
    int grid = (a.nlines + k->em_lines - 1) / k->em_lines;
    if (k->em_pipe && (fn == k->density || fn == k->density_store || fn == k->phase || fn == k->phase_real)) {
        const int pb = persistent_blocks((const void *)fn, k->em_threads());
        if (pb > 0 && pb < grid) grid = pb;
    }
    L.fn = (const void *)fn;
    L.grid = dim3(grid);
    L.block = dim3(k->em_threads());
    L.em = true;
    L.ea = a;
    L.pass = pass;
    return L;
}

// A persistent EM kernel outside the table: grid = resident blocks (at most
// one per tile).
static Launch em_launch_persistent(void (*fn)(EmArgs), const NKernels *k, const EmArgs &a, int pass)
{
    Launch L = em_launch(fn, k, a, pass);
    const int pb = persistent_blocks((const void *)fn, k->em_threads());
    if (pb > 0 && pb < (int)L.grid.x) L.grid = dim3(pb);
    return L;
}

static EmArgs em_base(gsn_grid g, float2 *psi)
{
    EmArgs a;
    std::memset(&a, 0, sizeof(a));
    a.psi = psi;
    a.half = g->half;
    a.nyq = g->nyq;
    a.tw = g->tw[g->ndim - 1];
    a.sct = g->sct;
    a.scale = 1.0;
    a.half2 = g->half2;
    a.nyq2 = g->nyq2;
    a.gam = g->fld_gamma;
    a.bet = g->fld_beta;
    a.vext = g->fld_V;
    if (g->local_on) {
        const double n = g->lp_n, fl = g->lp_floor;
        a.cp = g->lp_cp;
        a.pmode = g->lp_cp == 0.0 ? 0 : (n == 1.0 ? 1 : 2);
        a.pn1 = n - 1.0;
        a.pfac = a.pmode == 2 ? n / (n - 1.0) : 0.0;
        a.rfl = fl;
        a.sfl = std::sqrt(fl);
        a.cb2 = 0.5 * g->lp_cb;
        a.bohm = g->bohm_on ? 1 : 0;
        if (a.pmode == 1 && fl > 0.0) {
            a.f_fl = std::log(fl);
            a.F_fl = fl * (std::log(fl) - 1.0);
        } else if (a.pmode == 2 && fl > 0.0) {
            a.f_fl = a.pfac * std::pow(fl, n - 1.0);
            a.F_fl = std::pow(fl, n) / (n - 1.0);
        }
    }
    return a;
}

// K(0) of the grid's kernel: the contact and screened parts (the Newtonian
// k = 0 term is dropped); mY2 may be negative (Helmholtz, C > 0).
static double kernel_k0(gsn_grid g)
{
    double v = g->kern.c_contact;
    if (g->kern.c_yukawa != 0.0) v += g->kern.c_yukawa / g->mY2;
    return v;
}

// The kernel table of the grid's storage type.
static const NKernels *kfor(gsn_grid g, int N, int v)
{
    return g->storage == GSN_C128 ? kernels_for_c128(N, v) : kernels_for(N, v);
}

// Build every launch list from the current parameters (pointers never move).
static void build_core(gsn_grid g)
{
    const int nd = g->ndim, Nx = g->Nx, Ny = g->Ny, Nz = g->Nz;
    const int X = nd - 1, Y = nd - 2, Z = 0;   // table indices by axis
    const long long rows = g->P / Nx;
    const int H = Nx / 2;
    auto KX = [&](int pass) { return kfor(g, Nx, g->var[pass]); };
    // mass partials of the density pass (with the Bohm term: one per block)
    g->density_blocks = (int)((rows / 2 + KX(P_DENSITY)->em_lines - 1) / KX(P_DENSITY)->em_lines) *
                        (g->bohm_on ? 1 : KX(P_DENSITY)->em_parts);
    auto KY = [&](int pass) { return kfor(g, Ny, g->var[pass]); };
    auto KZ = [&](int pass) { return kfor(g, Nz, g->var[pass]); };
    g->entry.clear(); g->kin_half.clear(); g->kin_full.clear(); g->nonlin.clear();
    g->exit_.clear(); g->energy_rho.clear(); g->energy_kin.clear();

    // entry / exit along x
    {
        EmArgs a = em_base(g, g->psi);
        a.nlines = (int)rows;
        a.scale = 1.0;
        g->entry.push_back(em_launch(KX(P_ENTRY)->em_fwd, KX(P_ENTRY), a, P_ENTRY));
        a.scale = 1.0 / Nx;
        g->exit_.push_back(em_launch(KX(P_EXIT)->em_inv, KX(P_EXIT), a, P_EXIT));
    }
    // kinetic sub-steps (psi, full grid)
    for (int half = 0; half < 2; ++half) {
        std::vector<Launch> &dst = half ? g->kin_half : g->kin_full;
        double2 *const *kin = half ? g->kinH : g->kinF;
        if (nd == 3) {
            // the propagator exp(-i a |k|^2 h) is a product of per-axis
            // factors, so the kinetic sub-step is L_x L_y L_z with 1-D
            // operators that commute: one y pass applies
            // G_y exp(-i a (kx^2 + ky^2) h) F_y / Ny to the x-spectral psi
            // (kx per line), one z pass G_z exp(-i a kz^2 h) F_z / Nz
            const NKernels *ky = KY(P_KIN_Y), *kz = KZ(P_KINETIC);
            LmArgs a = lm_base(g, g->tw[Y], 1.0 / (double)Ny);
            a.s0 = make_seg(g->psi, Nx, 1, (long long)Ny * Nx, Nx, Nz, ky->lm_lines);
            a.s0.c1l = 1;  // c1 = x = line
            a.kin1 = kin[X];
            a.kinp = kin[Y];
            dst.push_back(lm_launch(ky->lm_kin, ky, a, P_KIN_Y));
            LmArgs b = lm_base(g, g->tw[Z], 1.0);
            b.s0 = make_seg(g->psi, (long long)Ny * Nx, 1, Nx, Nx, Ny, kz->lm_lines);
            b.kinp = kin[Z];
            b.kin_single = 1;
            dst.push_back(lm_launch(kz->lm_kin, kz, b, P_KINETIC));
        } else {
            const NKernels *ky = KY(P_KINETIC);
            LmArgs b = lm_base(g, g->tw[Y], 1.0 / (double)Ny);
            b.s0 = make_seg(g->psi, Nx, 1, 0, Nx, 1, ky->lm_lines);
            b.s0.c1l = 1;
            b.kin1 = kin[X];
            b.kinp = kin[Y];
            dst.push_back(lm_launch(ky->lm_kin, ky, b, P_KINETIC));
        }
    }
    // nonlinear sub-step
    const double K0 = kernel_k0(g);
    for (int energy = 0; energy < 2; ++energy) {
        std::vector<Launch> &dst = energy ? g->energy_rho : g->nonlin;
        float2 *src = energy ? g->scratch : g->psi;
        EmArgs d = em_base(g, src);
        d.nlines = (int)(rows / 2);
        d.partials = g->mass_parts;
        const bool store = g->store_psi && !energy;
        if (g->bohm_on) {
            const LKernels *lk = local_kernels_for(Nx, g->var[P_DENSITY]);
            if (!energy && lk->density_p[store ? 1 : 0])
                dst.push_back(em_launch_persistent(lk->density_p[store ? 1 : 0], KX(P_DENSITY), d, P_DENSITY));
            else
                dst.push_back(em_launch(store ? lk->density_store : lk->density, KX(P_DENSITY), d, P_DENSITY));
        } else {
            dst.push_back(em_launch(store ? KX(P_DENSITY)->density_store : KX(P_DENSITY)->density,
                                    KX(P_DENSITY), d, P_DENSITY));
        }
        if (g->fld_gamma || g->fld_beta) {
            // rho -> lap(rho) through the other axes, then the source pass
            if (g->fld_beta) {
                if (nd == 3) {
                    const NKernels *ky = KY(P_Y_FWD_SRC), *ky2 = KY(P_Y_INV_SRC);
                    const LKernels *lz = local_kernels_for(Nz, g->var[P_LAP_RHO]);
                    LmArgs e = lm_base(g, g->tw[Y], 1.0);
                    e.s0 = make_seg(g->half, H, 1, (long long)Ny * H, H, Nz, ky->lm_lines);
                    e.s1 = make_seg(g->nyq, 1, Ny, 0, Nz, 1, ky->lm_lines);
                    dst.push_back(lm_launch(ky->lm_fwd, ky, e, P_Y_FWD_SRC));
                    LmArgs f = lm_base(g, g->tw[Z], 0.5 / (double)g->P);
                    f.s0 = make_seg(g->half, (long long)Ny * H, 1, H, H, Ny, KZ(P_LAP_RHO)->lm_lines);
                    f.s0.c1l = 1;
                    f.s0.c2o = 1;
                    f.s1 = make_seg(g->nyq, Ny, 1, 0, Ny, 1, KZ(P_LAP_RHO)->lm_lines);
                    f.s1.c1f = H;
                    f.s1.c2l = 1;
                    f.k2_1 = g->k2[X];
                    f.k2_2 = g->k2[Y];
                    f.k2_p = g->k2[Z];
                    dst.push_back(lm_launch(lz->lm_lap, KZ(P_LAP_RHO), f, P_LAP_RHO));
                    LmArgs gg = lm_base(g, g->tw[Y], 1.0);
                    gg.s0 = make_seg(g->half, H, 1, (long long)Ny * H, H, Nz, ky2->lm_lines);
                    gg.s1 = make_seg(g->nyq, 1, Ny, 0, Nz, 1, ky2->lm_lines);
                    dst.push_back(lm_launch(ky2->lm_inv, ky2, gg, P_Y_INV_SRC));
                } else {
                    const LKernels *ly = local_kernels_for(Ny, g->var[P_LAP_RHO]);
                    LmArgs f = lm_base(g, g->tw[Y], 0.5 / (double)g->P);
                    f.s0 = make_seg(g->half, H, 1, 0, H, 1, KY(P_LAP_RHO)->lm_lines);
                    f.s0.c1l = 1;
                    f.s1 = make_seg(g->nyq, 1, 0, 0, 1, 1, KY(P_LAP_RHO)->lm_lines);
                    f.s1.c1f = H;
                    f.k2_1 = g->k2[X];
                    f.k2_p = g->k2[Y];
                    dst.push_back(lm_launch(ly->lm_lap, KY(P_LAP_RHO), f, P_LAP_RHO));
                }
            }
            EmArgs sa = em_base(g, src);
            sa.nlines = (int)(rows / 2);
            const LKernels *lk = local_kernels_for(Nx, g->var[P_SOURCE]);
            void (*sp)(EmArgs) = energy ? nullptr
                                        : lk->source_p[store ? 1 : 0][g->fld_beta ? 1 : 0][g->fld_gamma ? 1 : 0];
            if (sp)
                dst.push_back(em_launch_persistent(sp, KX(P_SOURCE), sa, P_SOURCE));
            else
                dst.push_back(em_launch(lk->source[store ? 1 : 0][g->fld_beta ? 1 : 0], KX(P_SOURCE), sa, P_SOURCE));
        }
        if (nd == 3) {
            const NKernels *ky = KY(P_Y_FWD_RHO), *kz = KZ(P_KERNEL), *ky2 = KY(P_Y_INV_PHI);
            LmArgs e = lm_base(g, g->tw[Y], 1.0);
            e.s0 = make_seg(g->half, H, 1, (long long)Ny * H, H, Nz, ky->lm_lines);
            e.s1 = make_seg(g->nyq, 1, Ny, 0, Nz, 1, ky->lm_lines);
            if (!energy) {
                e.reduce = 1;
                e.mass_parts = g->mass_parts;
                e.nmass = g->density_blocks;
                e.k0_dz_over_P = K0 * g->dz / (double)g->P;
            }
            dst.push_back(lm_launch(ky->lm_fwd, ky, e, P_Y_FWD_RHO));
            LmArgs f = lm_base(g, g->tw[Z], 1.0);
            f.s0 = make_seg(g->half, (long long)Ny * H, 1, H, H, Ny, kz->lm_lines);
            f.s0.c1l = 1;   // kx = line
            f.s0.c2o = 1;   // ky = outer
            f.s1 = make_seg(g->nyq, Ny, 1, 0, Ny, 1, kz->lm_lines);
            f.s1.c1f = H;   // kx = Nyquist
            f.s1.c2l = 1;   // ky = line
            f.k2_1 = g->k2[X];
            f.k2_2 = g->k2[Y];
            f.k2_p = g->k2[Z];
            set_kernel_args(g, f);
            dst.push_back(lm_launch(kz->lm_kern, kz, f, P_KERNEL));
            LmArgs gg = lm_base(g, g->tw[Y], 1.0);
            gg.s0 = make_seg(g->half, H, 1, (long long)Ny * H, H, Nz, ky2->lm_lines);
            gg.s1 = make_seg(g->nyq, 1, Ny, 0, Nz, 1, ky2->lm_lines);
            dst.push_back(lm_launch(ky2->lm_inv, ky2, gg, P_Y_INV_PHI));
        } else {
            const NKernels *ky = KY(P_KERNEL);
            LmArgs f = lm_base(g, g->tw[Y], 1.0);
            f.s0 = make_seg(g->half, H, 1, 0, H, 1, ky->lm_lines);
            f.s0.c1l = 1;
            f.s1 = make_seg(g->nyq, 1, 0, 0, 1, 1, ky->lm_lines);
            f.s1.c1f = H;
            f.k2_1 = g->k2[X];
            f.k2_p = g->k2[Y];
            set_kernel_args(g, f);
            if (!energy) {
                f.reduce = 1;
                f.mass_parts = g->mass_parts;
                f.nmass = g->density_blocks;
                f.k0_dz_over_P = K0 * g->dz / (double)g->P;
            }
            dst.push_back(lm_launch(ky->lm_kern, ky, f, P_KERNEL));
        }
        if (g->bohm_on) {
            // sqrt(rho) -> lap(sqrt rho): the same passes with -|k|^2 for K
            if (nd == 3) {
                const NKernels *ky = KY(P_Y_FWD_SQRT), *ky2 = KY(P_Y_INV_LAP);
                const LKernels *lz = local_kernels_for(Nz, g->var[P_LAPLACIAN]);
                LmArgs e = lm_base(g, g->tw[Y], 1.0);
                e.s0 = make_seg(g->half2, H, 1, (long long)Ny * H, H, Nz, ky->lm_lines);
                e.s1 = make_seg(g->nyq2, 1, Ny, 0, Nz, 1, ky->lm_lines);
                dst.push_back(lm_launch(ky->lm_fwd, ky, e, P_Y_FWD_SQRT));
                LmArgs f = lm_base(g, g->tw[Z], 0.5 / (double)g->P);
                f.s0 = make_seg(g->half2, (long long)Ny * H, 1, H, H, Ny, KZ(P_LAPLACIAN)->lm_lines);
                f.s0.c1l = 1;
                f.s0.c2o = 1;
                f.s1 = make_seg(g->nyq2, Ny, 1, 0, Ny, 1, KZ(P_LAPLACIAN)->lm_lines);
                f.s1.c1f = H;
                f.s1.c2l = 1;
                f.k2_1 = g->k2[X];
                f.k2_2 = g->k2[Y];
                f.k2_p = g->k2[Z];
                dst.push_back(lm_launch(lz->lm_lap, KZ(P_LAPLACIAN), f, P_LAPLACIAN));
                LmArgs gg = lm_base(g, g->tw[Y], 1.0);
                gg.s0 = make_seg(g->half2, H, 1, (long long)Ny * H, H, Nz, ky2->lm_lines);
                gg.s1 = make_seg(g->nyq2, 1, Ny, 0, Nz, 1, ky2->lm_lines);
                dst.push_back(lm_launch(ky2->lm_inv, ky2, gg, P_Y_INV_LAP));
            } else {
                const LKernels *ly = local_kernels_for(Ny, g->var[P_LAPLACIAN]);
                LmArgs f = lm_base(g, g->tw[Y], 0.5 / (double)g->P);
                f.s0 = make_seg(g->half2, H, 1, 0, H, 1, KY(P_LAPLACIAN)->lm_lines);
                f.s0.c1l = 1;
                f.s1 = make_seg(g->nyq2, 1, 0, 0, 1, 1, KY(P_LAPLACIAN)->lm_lines);
                f.s1.c1f = H;
                f.k2_1 = g->k2[X];
                f.k2_p = g->k2[Y];
                dst.push_back(lm_launch(ly->lm_lap, KY(P_LAPLACIAN), f, P_LAPLACIAN));
            }
        }
        EmArgs h = em_base(g, src);
        h.nlines = (int)(rows / 2);
        h.g = g->g;
        h.dz = g->dz;
        h.partials = g->epart;
        if (g->local_on || g->fld_V) {
            const LKernels *lk = local_kernels_for(Nx, g->var[P_PHASE]);
            void (*pp)(EmArgs) = energy ? nullptr : lk->phase_p[store ? 1 : 0][g->bohm_on ? 1 : 0][g->fld_V ? 1 : 0];
            if (pp)
                dst.push_back(em_launch_persistent(pp, KX(P_PHASE), h, P_PHASE));
            else
                dst.push_back(em_launch(energy ? lk->phase_energy : store ? lk->phase_real : lk->phase,
                                        KX(P_PHASE), h, P_PHASE));
        } else {
            dst.push_back(em_launch(energy ? KX(P_PHASE)->phase_energy
                                           : store ? KX(P_PHASE)->phase_real : KX(P_PHASE)->phase,
                                    KX(P_PHASE), h, P_PHASE));
        }
    }
    // kinetic energy: F_y (3-D) then the last-axis forward FFT with sum |k|^2 |psi_hat|^2
    {
        const int ep_off = 4 * g->max_density_blocks;
        if (nd == 3) {
            const NKernels *ky = KY(P_KIN_Y), *kz = KZ(P_KINETIC);
            LmArgs a = lm_base(g, g->tw[Y], 1.0);
            a.s0 = make_seg(g->scratch, Nx, 1, (long long)Ny * Nx, Nx, Nz, ky->lm_lines);
            g->energy_kin.push_back(lm_launch(ky->lm_fwd, ky, a, P_KIN_Y));
            LmArgs b = lm_base(g, g->tw[Z], 1.0);
            b.s0 = make_seg(g->scratch, (long long)Ny * Nx, 1, Nx, Nx, Ny, kz->lm_lines);
            b.s0.c1l = 1;
            b.s0.c2o = 1;
            b.k2_1 = g->k2[X];
            b.k2_2 = g->k2[Y];
            b.k2_p = g->k2[Z];
            b.partials = g->epart + ep_off;
            g->energy_kin.push_back(lm_launch(kz->lm_kin_energy, kz, b, P_KINETIC));
        } else {
            const NKernels *ky = KY(P_KINETIC);
            LmArgs b = lm_base(g, g->tw[Y], 1.0);
            b.s0 = make_seg(g->scratch, Nx, 1, 0, Nx, 1, ky->lm_lines);
            b.s0.c1l = 1;
            b.k2_1 = g->k2[X];
            b.k2_p = g->k2[Y];
            b.partials = g->epart + ep_off;
            g->energy_kin.push_back(lm_launch(ky->lm_kin_energy, ky, b, P_KINETIC));
        }
    }
}

// Every launch list: the fine step lists, the energy lists, the potential
// readout and (when a coarse ratio is set) the step lists of one coarse step,
// built by the same code with dz and the kinetic tables swapped.
static void build_schedule(gsn_grid g)
{
    build_core(g);
    if (g->coarse_ratio > 0) {
        StepLists fine{std::move(g->entry), std::move(g->kin_half), std::move(g->kin_full), std::move(g->nonlin),
                       std::move(g->exit_)};
        std::vector<Launch> er = std::move(g->energy_rho), ek = std::move(g->energy_kin);
        const double dz = g->dz;
        double2 *kf[3], *kh[3];
        for (int d = 0; d < 3; ++d) { kf[d] = g->kinF[d]; kh[d] = g->kinH[d]; }
        g->dz = dz * g->coarse_ratio;
        for (int d = 0; d < g->ndim; ++d) { g->kinF[d] = g->kinFc[d]; g->kinH[d] = g->kinHc[d]; }
        build_core(g);
        g->coarse = StepLists{std::move(g->entry), std::move(g->kin_half), std::move(g->kin_full),
                              std::move(g->nonlin), std::move(g->exit_)};
        g->dz = dz;
        for (int d = 0; d < 3; ++d) { g->kinF[d] = kf[d]; g->kinH[d] = kh[d]; }
        g->entry = std::move(fine.entry);
        g->kin_half = std::move(fine.kin_half);
        g->kin_full = std::move(fine.kin_full);
        g->nonlin = std::move(fine.nonlin);
        g->exit_ = std::move(fine.exit_);
        g->energy_rho = std::move(er);
        g->energy_kin = std::move(ek);
    }
    // potential readout of the real-space psi between calls: density straight
    // from real space (psi is only read), the potential passes, the C2R
    // readout kernel
    g->pot.clear();
    if (g->storage == GSN_C128) return;   // no potential readout on FP64-storage grids
    {
        const NKernels *kx = kernels_for(g->Nx, g->var[P_DENSITY]);
        EmArgs d = em_base(g, g->psi);
        d.nlines = (int)(g->P / g->Nx / 2);
        d.partials = g->mass_parts;
        g->pot.push_back(em_launch(kx->density_real, kx, d, P_DENSITY));
    }
    for (size_t i = 1; i + 1 < g->energy_rho.size(); ++i) {
        const int p = g->energy_rho[i].pass;
        if (p == P_Y_FWD_RHO || p == P_KERNEL || p == P_Y_INV_PHI) g->pot.push_back(g->energy_rho[i]);
    }
    {
        const NKernels *kx = kernels_for(g->Nx, g->var[P_PHASE]);
        EmArgs a = em_base(g, g->scratch);
        a.nlines = (int)(g->P / g->Nx / 2);
        g->pot.push_back(em_launch(kx->potential, kx, a, P_PHASE));
    }
    // the same readout taking x-spectral psi at the end of a coarse step: the
    // density pass that stores real-space psi back does the run's closing
    // inverse x transform and the density in one pass (not with the Bohm
    // term, whose density pass also transforms sqrt(rho))
    g->pot_spec.clear();
    if (!g->bohm_on && !g->pot.empty()) {
        const NKernels *kx = kernels_for(g->Nx, g->var[P_DENSITY]);
        EmArgs d = em_base(g, g->psi);
        d.nlines = (int)(g->P / g->Nx / 2);
        d.partials = g->mass_parts;
        g->pot_spec.push_back(em_launch(kx->density_store, kx, d, P_DENSITY));
        for (size_t i = 1; i < g->pot.size(); ++i) g->pot_spec.push_back(g->pot[i]);
    }
}

// With t0/t1 given, the two events are bound to the dispatch itself
// (hipExtLaunchKernel): they record the kernel's own start and end, and no
// marker is queued between this launch and its neighbours.
static hipError_t launch(const Launch &L, hipStream_t s, hipEvent_t t0 = nullptr, hipEvent_t t1 = nullptr)
{
    void *args[1];
    EmArgs ea = L.ea;
    LmArgs la = L.la;
    if (L.em) args[0] = &ea;
    else args[0] = &la;
    if (t0 || t1) return hipExtLaunchKernel(L.fn, L.grid, L.block, args, 0, s, t0, t1, 0);
    return hipLaunchKernel(L.fn, L.grid, L.block, args, 0, s);
}

static gsn_status run_list(gsn_grid g, const std::vector<Launch> &v)
{
    for (const Launch &L : v) HIP_TRY(launch(L, g->stream));
    return GSN_OK;
}

// ------------------------------------------------------------------ tables
// The tables are filled in a host copy of their part of the workspace and go to
// the device in one transfer (a 2-D grid took eleven at creation and four more
// with its coefficients, 15-20 us of waiting each).
template <class T> static T *host_of(gsn_grid g, T *dev) { return (T *)(g->tab.data() + ((char *)dev - g->tab_dev)); }

static gsn_status upload_tables(gsn_grid g)
{
    HIP_TRY(hipMemcpyAsync(g->tab_dev, g->tab.data(), g->tab.size(), hipMemcpyHostToDevice, g->stream));
    HIP_TRY(hipStreamSynchronize(g->stream));
    return GSN_OK;
}

// Read-outs land in a page of pinned host memory of the grid's own, so that they
// need no copy; where there is none (a grid in static memory, whose creation
// allocates nothing, or the allocation is refused) they go through the workspace.
// Allocated and freed in relaxed capture mode: another thread may be capturing.
static HostObs *alloc_obs()
{
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    const bool sw = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
    HostObs *p = nullptr;
    if (hipHostMalloc((void **)&p, sizeof(HostObs), hipHostMallocDefault) != hipSuccess) {
        (void)hipGetLastError();
        p = nullptr;
    }
    if (sw) (void)hipThreadExchangeStreamCaptureMode(&mode);
    return p;
}
static void free_obs(HostObs *p)
{
    if (!p) return;
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    const bool sw = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
    (void)hipHostFree(p);
    if (sw) (void)hipThreadExchangeStreamCaptureMode(&mode);
}

static void fill_kinetic(gsn_grid g, double dz, double2 *const *kf, double2 *const *kh)
{
    for (int d = 0; d < g->ndim; ++d) {
        const int N = g->n[d];
        double2 *f = host_of(g, kf[d]), *h = host_of(g, kh[d]);
        // the z pass has no other factor: its table holds the scale as well
        const double s = g->ndim == 3 && d == 0 ? 1.0 / N : 1.0;
        for (int j = 0; j < N; ++j) {
            const double k = wavenumber(j, N, g->L[d]);
            const double thf = -g->a * k * k * dz, thh = 0.5 * thf;
            f[j] = make_double2(s * std::cos(thf), s * std::sin(thf));
            h[j] = make_double2(s * std::cos(thh), s * std::sin(thh));
        }
    }
}

static gsn_status upload_kinetic(gsn_grid g)
{
    fill_kinetic(g, g->dz, g->kinF, g->kinH);
    if (g->coarse_ratio > 0) fill_kinetic(g, g->dz * g->coarse_ratio, g->kinFc, g->kinHc);
    return upload_tables(g);
}

static void fill_static_tables(gsn_grid g)
{
    for (int d = 0; d < g->ndim; ++d) {
        const int N = g->n[d];
        double2 *tw = host_of(g, g->tw[d]);
        double *k2 = host_of(g, g->k2[d]);
        for (int q = 0; q < N; ++q) {
            const double ang = 2.0 * M_PI * (double)q / (double)N;
            tw[q] = make_double2(std::cos(ang), -std::sin(ang));
            const double k = wavenumber(q, N, g->L[d]);
            k2[q] = k * k;
        }
    }
    fill_sincos_table(host_of(g, g->sct));
    *host_of(g, g->k2_unit) = 0.0;
    *host_of(g, g->kin_unit) = make_double2(1.0, 0.0);
}

// Schedule of a grid that has not been tuned.  Measured per step over the grids
// from 32^2 to 2048^2 and 32^3 to 512^3, plain, with local terms and with source
// fields, against e16 in every pass:
// - up to 2^19 points launches and their latencies bound a pass, not its
//   throughput: s4 (64x128 35 -> 17 us, 512^2 64 -> 28, 1024x512 69 -> 45,
//   32x256x64 64 -> 49; at 2^20 points 1024^2 takes 70 us with it and 69 with
//   p16).  The entry transform has one exchange less to wait for in s8 (64x2048
//   6.3 -> 6.0 us, 1024x512 5.3 -> 5.0, short lines equal); the exit stays with the
//   density pass, whose inverse transform takes its place in a corrected step;
// - above, p16: the plan of e16, so the same error (512^3 6735 -> 4202 us, 256^3
//   383 -> 332, 2048^2 242 -> 152; 128^3, the shape that gains least, 86 -> 88).
//   p8 is up to a quarter faster (512^3 3460 us, 2048^2 131, 128x128x64 59 against
//   71), but its plan exchanges, and rounds to complex64, more often on lines of 16,
//   128, 256, 1024 and 2048 points: psi is 3% to 37% further off 64 bits, and 5%
//   where only one axis has 512 points.  Tuning may choose it, a first schedule not;
// - complex128 grids above 2^19 points keep e16: their persistent passes are the
//   one-tile passes (256^3 567 us, e8 613).
constexpr long long kLatencyPoints = 1LL << 19;
static int default_variant(gsn_grid g, int pass)
{
    enum { E16 = 0, P16 = 2, S8 = 4 };
    if (g->P <= kLatencyPoints) return pass == P_ENTRY ? S8 : kSmallVariant;
    return g->storage == GSN_C128 ? E16 : P16;
}

// ------------------------------------------------------------------ lifecycle
static gsn_status create_grid(gsn_grid *out, int ndim, const int32_t n[], const double L[], int storage,
                              void *d_workspace, size_t bytes, void *hip_stream, bool static_ws)
{
    if (!out) return fail(GSN_EINVAL, "out is NULL");
    if (storage != GSN_C64 && storage != GSN_C128) {
        *out = nullptr;
        return fail(GSN_EINVAL, "storage must be GSN_C64 or GSN_C128");
    }
    *out = nullptr;
    gsn_status s = validate_shape(ndim, n);
    if (s) return s;
    if (!L) return fail(GSN_EINVAL, "L is NULL");
    for (int d = 0; d < ndim; ++d)
        if (!(std::isfinite(L[d]) && L[d] > 0.0)) return fail(GSN_EINVAL, "box lengths must be finite and > 0");
    if (!d_workspace) return fail(GSN_EINVAL, "workspace is NULL");
    if (((uintptr_t)d_workspace & 255) != 0) return fail(GSN_EWORKSPACE, "workspace must be 256-byte aligned");
    const Layout lay = compute_layout(ndim, n, storage_bytes(storage));
    if (bytes < lay.total)
        return fail(GSN_EWORKSPACE, "workspace too small: need " + std::to_string(lay.total) + " bytes");

    gsn_grid g = new (std::nothrow) gsn_grid_();
    if (!g) return fail(GSN_EINVAL, "out of host memory");
    g->storage = storage;
    g->esz = storage_bytes(storage);
    g->ndim = ndim;
    for (int d = 0; d < 3; ++d) { g->n[d] = d < ndim ? n[d] : 1; g->L[d] = d < ndim ? L[d] : 1.0; }
    g->Nx = n[ndim - 1];
    g->Ny = n[ndim - 2];
    g->Nz = ndim == 3 ? n[0] : 1;
    g->P = (long long)g->Nx * g->Ny * g->Nz;
    g->stream = (hipStream_t)hip_stream;
    for (int i = 0; i < P_COUNT; ++i) g->var[i] = default_variant(g, i);
    g->store_psi = 0;
    g->max_density_blocks = lay.density_blocks;
    g->a = 0.5;
    g->g = 0.0;
    g->dz = 0.0;
    std::memset(&g->kern, 0, sizeof(g->kern));
    g->mY2 = 0.0;
    g->lp_cp = g->lp_cb = g->lp_floor = 0.0;
    g->lp_n = 1.0;
    g->local_on = g->bohm_on = false;
    g->fld_gamma = g->fld_beta = g->fld_V = nullptr;
    if (hipGetDevice(&g->device) != hipSuccess) {
        delete g;
        return fail(GSN_EHIP, "hipGetDevice failed");
    }
    char *ws = (char *)d_workspace;
    g->psi = (float2 *)(ws + lay.psi);
    g->scratch = (float2 *)(ws + lay.scratch);
    g->half = (float2 *)(ws + lay.half);
    g->nyq = (float2 *)(ws + lay.nyq);
    g->half2 = (float2 *)(ws + lay.half2);
    g->nyq2 = (float2 *)(ws + lay.nyq2);
    g->mass_parts = (double *)(ws + lay.mass_parts);
    g->epart = (double *)(ws + lay.epart);
    g->st = (DevState *)(ws + lay.st);
    size_t off = lay.tables;
    for (int d = 0; d < ndim; ++d) {
        g->tw[d] = (double2 *)(ws + off); off += align256(16ull * n[d]);
        g->kinF[d] = (double2 *)(ws + off); off += align256(16ull * n[d]);
        g->kinH[d] = (double2 *)(ws + off); off += align256(16ull * n[d]);
        g->k2[d] = (double *)(ws + off); off += align256(8ull * n[d]);
        g->kinFc[d] = (double2 *)(ws + off); off += align256(16ull * n[d]);
        g->kinHc[d] = (double2 *)(ws + off); off += align256(16ull * n[d]);
    }
    g->k2_unit = (double *)(ws + off); off += 256;
    g->kin_unit = (double2 *)(ws + off); off += 256;
    g->st_save[0] = (DevState *)(ws + off); off += 256;
    g->st_save[1] = (DevState *)(ws + off); off += 256;
    g->sct = (double2 *)(ws + off); off += 16 * kSinCosTable;
    g->coarse_ratio = 0;
    g->static_ws = static_ws;
    g->tab_dev = ws + lay.tables;
    try {
        g->tab.assign(lay.total - lay.tables, 0);
    } catch (const std::bad_alloc &) {
        delete g;
        return fail(GSN_EINVAL, "out of host memory");
    }
    g->obs_dev = (HostObs *)(ws + lay.obs);
    g->obs_host = nullptr;
    fill_static_tables(g);
    if ((s = upload_kinetic(g))) {
        delete g;
        return s;
    }
    hipLaunchKernelGGL(k_reset_state, dim3(1), dim3(64), 0, g->stream, g->st);
    if (hipGetLastError() != hipSuccess) {
        delete g;
        return fail(GSN_EHIP, "reset kernel launch failed");
    }
    if (!static_ws) g->obs_host = alloc_obs();
    build_schedule(g);
    *out = g;
    return GSN_OK;
}

extern "C" gsn_status gsn_create_ex(gsn_grid *out, int ndim, const int32_t n[], const double L[], int storage,
                                    void *d_workspace, size_t bytes, void *hip_stream)
{
    return create_grid(out, ndim, n, L, storage, d_workspace, bytes, hip_stream, false);
}

extern "C" gsn_status gsn_create(gsn_grid *out, int ndim, const int32_t n[], const double L[],
                                 void *d_workspace, size_t bytes, void *hip_stream)
{
    return gsn_create_ex(out, ndim, n, L, GSN_C64, d_workspace, bytes, hip_stream);
}

// ------------------------------------------------------------------ grids without a caller workspace
// For callers that cannot allocate device memory (code under HIP graph
// capture, serving loops, harnesses that forbid hipMalloc): a grid whose
// workspace is this file-scope array.  Every GPU the library runs on holds its
// own copy until the process ends.  In host code the array's name is only a
// host-side stand-in; its device address on the current device comes from
// hipGetSymbolAddress, taken once per device and kept in g_static_ws.
constexpr size_t kStaticWorkspaceBytes = 64ull << 20;
static __device__ __align__(256) unsigned char scratch[kStaticWorkspaceBytes];

namespace {
struct StaticWs {
    void *ptr = nullptr;   // device address of scratch on this device
    bool in_use = false;   // a live grid owns it
};
std::mutex g_static_mu;
std::map<int, StaticWs> g_static_ws;
}  // namespace

extern "C" gsn_status gsn_create_static(gsn_grid *out, int ndim, const int32_t n[], const double L[],
                                        void *hip_stream)
{
    if (!out) return fail(GSN_EINVAL, "out is NULL");
    *out = nullptr;
    gsn_status s = validate_shape(ndim, n);
    if (s) return s;
    const Layout lay = compute_layout(ndim, n, storage_bytes(GSN_C64));
    if (lay.total > kStaticWorkspaceBytes)
        return fail(GSN_EWORKSPACE, "grid needs " + std::to_string(lay.total) +
                                        " bytes of workspace; the static workspace holds " +
                                        std::to_string(kStaticWorkspaceBytes));
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lock(g_static_mu);
    StaticWs &w = g_static_ws[dev];
    if (!w.ptr) {
        void *ptr = nullptr;
        HIP_TRY(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        if (!ptr) return fail(GSN_EHIP, "hipGetSymbolAddress returned no address for the static workspace");
        w.ptr = ptr;
    }
    if (w.in_use) return fail(GSN_ESTATE, "the static workspace of this device belongs to a live grid");
    gsn_grid g = nullptr;
    if ((s = create_grid(&g, ndim, n, L, GSN_C64, w.ptr, kStaticWorkspaceBytes, hip_stream, true))) return s;
    w.in_use = true;
    *out = g;
    return GSN_OK;
}

extern "C" gsn_status gsn_destroy(gsn_grid g)
{
    if (!g) return fail(GSN_EINVAL, "grid is NULL");
    (void)hipStreamSynchronize(g->stream);
    free_obs(g->obs_host);
    if (g->static_ws) {
        std::lock_guard<std::mutex> lock(g_static_mu);
        g_static_ws[g->device].in_use = false;
    }
    delete g;
    return GSN_OK;
}

extern "C" gsn_status gsn_set_kernel(gsn_grid g, const gsn_kernel *k)
{
    if (!g || !k) return fail(GSN_EINVAL, "NULL argument");
    if (!std::isfinite(k->c_newton) || !std::isfinite(k->c_yukawa) || !std::isfinite(k->m_yukawa) ||
        !std::isfinite(k->c_contact))
        return fail(GSN_EINVAL, "kernel coefficients must be finite");
    if (k->c_yukawa != 0.0 && !(k->m_yukawa > 0.0))
        return fail(GSN_EINVAL, "m_yukawa must be > 0 when c_yukawa != 0");
    g->kern = *k;
    g->mY2 = k->m_yukawa * k->m_yukawa;
    build_schedule(g);
    return GSN_OK;
}

// Whether some grid wavenumber has |k|^2 = C (relative tolerance 1e-12): the
// per-axis |k_d|^2 values are sorted, and for every combination of the other
// axes the remainder is looked up in the last axis.
static bool resonant(gsn_grid g, double C)
{
    if (!(C > 0.0)) return false;
    std::vector<std::vector<double>> ks(g->ndim);
    for (int d = 0; d < g->ndim; ++d) {
        for (int j = 0; j <= g->n[d] / 2; ++j) {
            const double k = wavenumber(j, g->n[d], g->L[d]);
            ks[d].push_back(k * k);
        }
        std::sort(ks[d].begin(), ks[d].end());
    }
    const double tol = 1e-12 * std::max(1.0, C);
    const std::vector<double> &last = ks[g->ndim - 1];
    auto hit = [&](double target) {
        auto it = std::lower_bound(last.begin(), last.end(), target - tol);
        return it != last.end() && *it <= target + tol;
    };
    if (g->ndim == 2) {
        for (double a : ks[0])
            if (hit(C - a)) return true;
    } else {
        for (double a : ks[0])
            for (double b : ks[1])
                if (hit(C - a - b)) return true;
    }
    return false;
}

extern "C" gsn_status gsn_set_equation(gsn_grid g, double A, double B, double C, double D)
{
    if (!g) return fail(GSN_EINVAL, "grid is NULL");
    if (!std::isfinite(A) || !std::isfinite(B) || !std::isfinite(C) || !std::isfinite(D))
        return fail(GSN_EINVAL, "A, B, C, D must be finite");
    if (resonant(g, C))
        return fail(GSN_EINVAL, "C equals |k|^2 of a grid wavenumber: Eq. (2) has no periodic solution");
    HIP_TRY(hipSetDevice(g->device));
    HIP_TRY(hipStreamSynchronize(g->stream));
    std::memset(&g->kern, 0, sizeof(g->kern));
    if (C == 0.0) {
        g->kern.c_newton = B * D;
        g->mY2 = 0.0;
    } else {
        g->kern.c_yukawa = B * D;
        g->kern.m_yukawa = std::sqrt(std::fabs(C));
        g->mY2 = -C;
    }
    g->a = -A;
    if (g->have_dz) {
        gsn_status s = upload_kinetic(g);
        if (s) return s;
    }
    build_schedule(g);
    return GSN_OK;
}

extern "C" gsn_status gsn_set_local_terms(gsn_grid g, double c_pressure, double n_pressure, double c_bohm,
                                          double rho_floor)
{
    if (!g) return fail(GSN_EINVAL, "grid is NULL");
    if (!std::isfinite(c_pressure) || !std::isfinite(n_pressure) || !std::isfinite(c_bohm) ||
        !std::isfinite(rho_floor))
        return fail(GSN_EINVAL, "local-term coefficients must be finite");
    if (rho_floor < 0.0) return fail(GSN_EINVAL, "rho_floor must be >= 0");
    if (c_pressure != 0.0 && n_pressure >= 0.0 && n_pressure < 1.0)
        return fail(GSN_EINVAL, "the pressure law is defined for n = 1, n > 1 and n < 0");
    if (((c_pressure != 0.0 && n_pressure <= 1.0) || c_bohm != 0.0) && !(rho_floor > 0.0))
        return fail(GSN_EINVAL, "ln rho, negative powers of rho and the Bohm term need rho_floor > 0");
    if (g->storage == GSN_C128 && (c_pressure != 0.0 || c_bohm != 0.0))
        return fail(GSN_EUNSUPPORTED, "the Eq. (15) local terms run on complex64 grids");
    HIP_TRY(hipSetDevice(g->device));
    HIP_TRY(hipStreamSynchronize(g->stream));
    g->lp_cp = c_pressure;
    g->lp_n = n_pressure;
    g->lp_cb = c_bohm;
    g->lp_floor = rho_floor;
    g->local_on = c_pressure != 0.0 || c_bohm != 0.0;
    g->bohm_on = c_bohm != 0.0;
    build_schedule(g);
    return GSN_OK;
}

extern "C" gsn_status gsn_set_source_fields(gsn_grid g, const float *gamma, const float *beta, const float *V_ext,
                                            size_t count)
{
    if (!g) return fail(GSN_EINVAL, "grid is NULL");
    if ((gamma || beta || V_ext) && count != (size_t)g->P)
        return fail(GSN_EINVAL, "each field must hold exactly P = " + std::to_string(g->P) + " values");
    if (g->storage == GSN_C128 && (gamma || beta || V_ext))
        return fail(GSN_EUNSUPPORTED, "source fields run on complex64 grids");
    HIP_TRY(hipSetDevice(g->device));
    HIP_TRY(hipStreamSynchronize(g->stream));
    g->fld_gamma = gamma;
    g->fld_beta = beta;
    g->fld_V = V_ext;
    build_schedule(g);
    return GSN_OK;
}

extern "C" gsn_status gsn_nmc_fields(gsn_grid g, double lambda, double r0, double nu, const double *center,
                                     double r_min, float *gamma, float *beta, float *V_ext, size_t count)
{
    if (!g) return fail(GSN_EINVAL, "grid is NULL");
    if (count < (size_t)g->P) return fail(GSN_EINVAL, "outputs must hold P = " + std::to_string(g->P) + " values");
    if (!(std::isfinite(lambda) && lambda > 0.0) || !(std::isfinite(r0) && r0 > 0.0) || !std::isfinite(nu) ||
        nu == 0.0 || !(std::isfinite(r_min) && r_min > 0.0))
        return fail(GSN_EINVAL, "need lambda > 0, r0 > 0, nu != 0 and r_min > 0, all finite");
    double c[3] = {0.0, 0.0, 0.0};
    if (center)
        for (int d = 0; d < g->ndim; ++d) {
            if (!std::isfinite(center[d])) return fail(GSN_EINVAL, "centre must be finite");
            c[d] = center[d];
        }
    HIP_TRY(hipSetDevice(g->device));
    HIP_TRY(launch_nmc_fields(g->ndim, g->n, g->L, c, lambda, r0, nu, r_min, gamma, beta, V_ext, g->stream));
    HIP_TRY(hipStreamSynchronize(g->stream));
    return GSN_OK;
}

extern "C" gsn_status gsn_set_coefficients(gsn_grid g, double a_kin, double g_local, double dz)
{
    if (!g) return fail(GSN_EINVAL, "grid is NULL");
    if (!std::isfinite(a_kin) || !std::isfinite(g_local) || !std::isfinite(dz) || dz == 0.0)
        return fail(GSN_EINVAL, "coefficients must be finite and dz != 0");
    HIP_TRY(hipSetDevice(g->device));
    HIP_TRY(hipStreamSynchronize(g->stream));
    g->a = a_kin;
    g->g = g_local;
    g->dz = dz;
    gsn_status s = upload_kinetic(g);
    if (s) return s;
    g->have_dz = true;
    build_schedule(g);
    return GSN_OK;
}

extern "C" gsn_status gsn_set_psi(gsn_grid g, const void *src, int on_device, int dtype)
{
    if (!g || !src) return fail(GSN_EINVAL, "NULL argument");
    if (dtype != GSN_C64 && dtype != GSN_C128) return fail(GSN_EINVAL, "dtype must be GSN_C64 or GSN_C128");
    HIP_TRY(hipSetDevice(g->device));
    const long long P = g->P;
    if (g->storage == GSN_C128) {
        if (dtype == GSN_C128) {
            HIP_TRY(hipMemcpyAsync(g->psi, src, 16ull * P, on_device ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice,
                                   g->stream));
        } else if (on_device) {
            HIP_TRY(launch_from_c64(src, g->psi, P, g->stream));
        } else {
            std::vector<double2> tmp((size_t)P);
            const float *s = (const float *)src;
            for (long long i = 0; i < P; ++i) tmp[i] = make_double2((double)s[2 * i], (double)s[2 * i + 1]);
            HIP_TRY(hipMemcpyAsync(g->psi, tmp.data(), 16ull * P, hipMemcpyHostToDevice, g->stream));
            HIP_TRY(hipStreamSynchronize(g->stream));
        }
    } else if (dtype == GSN_C64) {
        HIP_TRY(hipMemcpyAsync(g->psi, src, 8ull * P, on_device ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice,
                               g->stream));
    } else if (on_device) {
        hipLaunchKernelGGL(k_from_c128, dim3(1024), dim3(256), 0, g->stream, (const double2 *)src, g->psi, P);
        HIP_TRY(hipGetLastError());
    } else {
        std::vector<float2> tmp((size_t)P);
        const double *s = (const double *)src;
        for (long long i = 0; i < P; ++i) tmp[i] = make_float2((float)s[2 * i], (float)s[2 * i + 1]);
        HIP_TRY(hipMemcpyAsync(g->psi, tmp.data(), 8ull * P, hipMemcpyHostToDevice, g->stream));
        HIP_TRY(hipStreamSynchronize(g->stream));
    }
    hipLaunchKernelGGL(k_reset_state, dim3(1), dim3(64), 0, g->stream, g->st);
    HIP_TRY(hipGetLastError());
    if (!on_device) HIP_TRY(hipStreamSynchronize(g->stream));
    g->have_psi = true;
    return GSN_OK;
}

static gsn_status ready(gsn_grid g)
{
    if (!g) return fail(GSN_EINVAL, "grid is NULL");
    if (!g->have_psi) return fail(GSN_ESTATE, "psi not set");
    if (!g->have_dz) return fail(GSN_ESTATE, "coefficients (dz) not set");
    if ((g->fld_gamma || g->fld_beta) && kernel_k0(g) != 0.0)
        return fail(GSN_EUNSUPPORTED, "source fields need a kernel with K(0) = 0 (no screened or contact part)");
    return GSN_OK;
}

extern "C" gsn_status gsn_step(gsn_grid g, int64_t nsteps)
{
    gsn_status s = ready(g);
    if (s) return s;
    if (nsteps < 0) return fail(GSN_EINVAL, "nsteps must be >= 0");
    if (nsteps == 0) return GSN_OK;
    HIP_TRY(hipSetDevice(g->device));
    if ((s = run_list(g, g->entry)) || (s = run_list(g, g->kin_half))) return s;
    for (int64_t i = 0; i < nsteps; ++i) {
        if ((s = run_list(g, g->nonlin))) return s;
        if ((s = run_list(g, i + 1 < nsteps ? g->kin_full : g->kin_half))) return s;
    }
    return run_list(g, g->exit_);
}

// Queue the sums of the given columns (and the state) and wait for them: one
// launch that writes to host memory and one wait, where a read of each column
// by itself took a copy and a wait of 15-20 us apiece (an energy 172 us).
static gsn_status read_obs(gsn_grid g, const ObsArgs &cols, HostObs *out)
{
    HostObs *dst = g->obs_host ? g->obs_host : g->obs_dev;
    // the launch's own status: the thread's last error may be another library's
    ObsArgs c = cols;
    void *args[] = {&c, &g->st, &dst};
    HIP_TRY(hipLaunchKernel((const void *)k_obs, dim3(cols.ncol + 1), dim3(256), args, 0, g->stream));
    if (!g->obs_host) HIP_TRY(hipMemcpyAsync(out, dst, sizeof(HostObs), hipMemcpyDeviceToHost, g->stream));
    HIP_TRY(hipStreamSynchronize(g->stream));
    if (g->obs_host) *out = *g->obs_host;
    return GSN_OK;
}

static gsn_status check_state(const DevState &st)
{
    if (st.nonfinite) return fail(GSN_ENONFINITE, "the fused FP64 mass became non-finite");
    return GSN_OK;
}

static gsn_status read_state(gsn_grid g, DevState *st)
{
    HostObs o;
    gsn_status s = read_obs(g, ObsArgs{}, &o);
    if (s) return s;
    *st = o.st;
    return GSN_OK;
}

extern "C" gsn_status gsn_sync(gsn_grid g)
{
    if (!g) return fail(GSN_EINVAL, "grid is NULL");
    HIP_TRY(hipSetDevice(g->device));
    DevState st;
    gsn_status s = read_state(g, &st);
    if (s) return s;
    return check_state(st);
}

extern "C" gsn_status gsn_phase(gsn_grid g, double *theta, int64_t *steps)
{
    if (!g) return fail(GSN_EINVAL, "grid is NULL");
    HIP_TRY(hipSetDevice(g->device));
    DevState st;
    gsn_status s = read_state(g, &st);
    if (s) return s;
    if (theta) *theta = st.theta;
    if (steps) *steps = st.steps;
    return GSN_OK;
}

extern "C" gsn_status gsn_get_psi(gsn_grid g, void *dst, int on_device, int dtype)
{
    if (!g || !dst) return fail(GSN_EINVAL, "NULL argument");
    if (dtype != GSN_C64 && dtype != GSN_C128) return fail(GSN_EINVAL, "dtype must be GSN_C64 or GSN_C128");
    if (!g->have_psi) return fail(GSN_ESTATE, "psi not set");
    HIP_TRY(hipSetDevice(g->device));
    const long long P = g->P;
    if (g->storage == GSN_C128) {
        // through the scratch buffer (16 bytes per point) in chunks
        const size_t osz = dtype == GSN_C128 ? 16 : 8;
        const long long chunk = on_device ? P : (long long)((16ull * P) / osz);
        for (long long off = 0; off < P; off += chunk) {
            const long long cnt = P - off < chunk ? P - off : chunk;
            const double2 *src = (const double2 *)g->psi + off;
            if (on_device) {
                HIP_TRY(launch_readout_c128(src, dst, dtype == GSN_C128, cnt, g->st, g->stream));
            } else {
                HIP_TRY(launch_readout_c128(src, g->scratch, dtype == GSN_C128, cnt, g->st, g->stream));
                HIP_TRY(hipMemcpyAsync((char *)dst + off * osz, g->scratch, cnt * osz, hipMemcpyDeviceToHost,
                                       g->stream));
                HIP_TRY(hipStreamSynchronize(g->stream));
            }
        }
        return gsn_sync(g);
    }
    if (on_device) {
        if (dtype == GSN_C128) hipLaunchKernelGGL(k_readout<true>, dim3(1024), dim3(256), 0, g->stream, g->psi, dst, P, g->st);
        else hipLaunchKernelGGL(k_readout<false>, dim3(1024), dim3(256), 0, g->stream, g->psi, dst, P, g->st);
        HIP_TRY(hipGetLastError());
    } else {
        // through the scratch buffer (8 bytes per point) in chunks
        const size_t esz = dtype == GSN_C128 ? 16 : 8;
        const long long chunk = (long long)((8ull * P) / esz);
        for (long long off = 0; off < P; off += chunk) {
            const long long cnt = P - off < chunk ? P - off : chunk;
            if (dtype == GSN_C128)
                hipLaunchKernelGGL(k_readout<true>, dim3(1024), dim3(256), 0, g->stream, g->psi + off,
                                   (void *)g->scratch, cnt, g->st);
            else
                hipLaunchKernelGGL(k_readout<false>, dim3(1024), dim3(256), 0, g->stream, g->psi + off,
                                   (void *)g->scratch, cnt, g->st);
            HIP_TRY(hipGetLastError());
            HIP_TRY(hipMemcpyAsync((char *)dst + off * esz, g->scratch, cnt * esz, hipMemcpyDeviceToHost,
                                   g->stream));
            HIP_TRY(hipStreamSynchronize(g->stream));
        }
    }
    return gsn_sync(g);
}

static double cell_volume(gsn_grid g)
{
    double dV = 1.0;
    for (int d = 0; d < g->ndim; ++d) dV *= g->L[d] / g->n[d];
    return dV;
}

extern "C" gsn_status gsn_mass(gsn_grid g, double *mass)
{
    if (!mass) return fail(GSN_EINVAL, "mass is NULL");
    gsn_status s = g ? GSN_OK : fail(GSN_EINVAL, "grid is NULL");
    if (s) return s;
    if (!g->have_psi) return fail(GSN_ESTATE, "psi not set");
    HIP_TRY(hipSetDevice(g->device));
    const int nb = 1024;
    if (g->storage == GSN_C128) {
        HIP_TRY(launch_mass_c128(g->psi, g->P, g->epart, nb, g->stream));
    } else {
        hipLaunchKernelGGL(k_mass<256>, dim3(nb), dim3(256), 0, g->stream, g->psi, g->P, g->epart);
        HIP_TRY(hipGetLastError());
    }
    // summed here, in the order in which the batch sums its instances' partials
    ObsArgs cols{};
    cols.add(g->epart, nb, 1);
    cols.raw = nb;
    HostObs o;
    if ((s = read_obs(g, cols, &o))) return s;
    double sum = 0.0;
    for (int i = 0; i < nb; ++i) sum += o.raw[i];
    *mass = sum * cell_volume(g);
    if ((s = check_state(o.st))) return s;
    if (!std::isfinite(*mass)) return fail(GSN_ENONFINITE, "mass is not finite");
    return GSN_OK;
}

extern "C" gsn_status gsn_energy(gsn_grid g, double e[4])
{
    if (!e) return fail(GSN_EINVAL, "e is NULL");
    gsn_status s = g ? GSN_OK : fail(GSN_EINVAL, "grid is NULL");
    if (s) return s;
    if (g->fld_gamma || g->fld_beta)
        return fail(GSN_EUNSUPPORTED, "no energy with position-dependent source fields");
    if (!g->have_psi) return fail(GSN_ESTATE, "psi not set");
    HIP_TRY(hipSetDevice(g->device));
    HIP_TRY(hipMemcpyAsync(g->scratch, g->psi, g->esz * g->P, hipMemcpyDeviceToDevice, g->stream));
    for (const Launch &L : g->entry) {
        Launch c = L;
        c.ea.psi = g->scratch;
        HIP_TRY(launch(c, g->stream));
    }
    if ((s = run_list(g, g->energy_rho))) return s;
    if ((s = run_list(g, g->energy_kin))) return s;
    const int nphase = (int)g->energy_rho.back().grid.x;
    const int nkin = (int)g->energy_kin.back().grid.x;
    ObsArgs cols{};
    cols.add(g->mass_parts, g->density_blocks, 1);
    for (int c = 0; c < 4; ++c) cols.add(g->epart + c, nphase, 4);
    cols.add(g->epart + 4 * g->max_density_blocks, nkin, 1);
    HostObs o;
    if ((s = read_obs(g, cols, &o))) return s;
    const double rho_sum = o.v[0], rho_phi = o.v[1], rho2 = o.v[2], gsum = o.v[3], slap = o.v[4], k2sum = o.v[5];
    const double dV = cell_volume(g), P = (double)g->P, K0 = kernel_k0(g);
    const double ekin = g->a * dV / P * k2sum;
    // Kerr, pressure and static potential (-sum (c_p G + V rho)) and Bohm
    // (-(c_B/2) sum s lap s = (c_B/2) sum |grad s|^2)
    const double eloc = -0.5 * g->g * dV * rho2 - dV * gsum - 0.5 * g->lp_cb * dV * slap;
    const double enl = -0.5 * dV * (rho_phi + K0 * rho_sum * rho_sum / P);
    e[0] = ekin + eloc + enl;
    e[1] = ekin;
    e[2] = eloc;
    e[3] = enl;
    return check_state(o.st);
}

// ------------------------------------------------------------------ profiling
extern "C" int gsn_pass_count(gsn_grid) { return P_COUNT; }

extern "C" const char *gsn_pass_name(gsn_grid, int i)
{
    return (i >= 0 && i < P_COUNT) ? kPassNames[i] : "";
}

static double pass_bytes_c64(gsn_grid g, int i);

extern "C" double gsn_pass_bytes_per_point(gsn_grid g, int i)
{
    if (!g) return 0.0;
    // the model is written for complex64 values; FP64 storage doubles every byte
    return pass_bytes_c64(g, i) * (double)(g->esz / 8);
}

static double pass_bytes_c64(gsn_grid g, int i)
{
    // reads + writes of complex64 psi (8 B), half spectrum (4 B per point)
    switch (i) {
    case P_ENTRY: case P_EXIT: case P_KINETIC: return 16.0;
    case P_KIN_Y: return g->ndim == 3 ? 16.0 : 0.0;
    case P_DENSITY: return (g->store_psi ? 20.0 : 12.0) + (g->bohm_on ? 4.0 : 0.0);
    case P_Y_FWD_RHO: case P_KERNEL: case P_Y_INV_PHI: return 8.0;
    case P_PHASE: return 20.0 + (g->bohm_on ? 4.0 : 0.0) + (g->fld_V ? 4.0 : 0.0);
    case P_Y_FWD_SQRT: case P_Y_INV_LAP: return g->bohm_on && g->ndim == 3 ? 8.0 : 0.0;
    case P_LAPLACIAN: return g->bohm_on ? 8.0 : 0.0;
    case P_Y_FWD_SRC: case P_Y_INV_SRC: return g->fld_beta && g->ndim == 3 ? 8.0 : 0.0;
    case P_LAP_RHO: return g->fld_beta ? 8.0 : 0.0;
    case P_SOURCE:
        if (!(g->fld_gamma || g->fld_beta)) return 0.0;
        // psi in, s spectrum out, lap(rho) spectrum and fields in
        return 12.0 + (g->fld_beta ? 8.0 : 0.0) + (g->fld_gamma ? 4.0 : 0.0);
    default: return 0.0;
    }
}

extern "C" gsn_status gsn_profile_passes(gsn_grid g, int64_t nsteps, double *ms, int npass)
{
    gsn_status s = ready(g);
    if (s) return s;
    if (!ms || npass < P_COUNT || nsteps < 1) return fail(GSN_EINVAL, "bad profile arguments");
    HIP_TRY(hipSetDevice(g->device));
    // a start and a stop event per launch in flight, kChunk launches between
    // synchronisations (so any nsteps needs a fixed number of events),
    // destroyed on every return path
    constexpr size_t kChunk = 256;
    struct Events {
        std::vector<hipEvent_t> ev;
        ~Events()
        {
            for (hipEvent_t e : ev)
                if (e) (void)hipEventDestroy(e);
        }
    } E;
    E.ev.assign(2 * kChunk, nullptr);
    for (auto &e : E.ev) HIP_TRY(hipEventCreate(&e));
    std::vector<double> tot(P_COUNT, 0.0);
    std::vector<long long> cnt(P_COUNT, 0);
    std::vector<int> pend;   // pass of each launch since the last synchronisation
    pend.reserve(kChunk);
    auto harvest = [&]() -> hipError_t {
        hipError_t e = hipStreamSynchronize(g->stream);
        for (size_t j = 0; e == hipSuccess && j < pend.size(); ++j) {
            float t = 0.f;
            e = hipEventElapsedTime(&t, E.ev[2 * j], E.ev[2 * j + 1]);
            tot[pend[j]] += t;
            cnt[pend[j]] += 1;
        }
        pend.clear();
        return e;
    };
    auto timed = [&](const Launch &L) -> hipError_t {
        const size_t j = pend.size();
        const hipError_t e = launch(L, g->stream, E.ev[2 * j], E.ev[2 * j + 1]);
        if (e != hipSuccess) return e;
        pend.push_back(L.pass);
        return pend.size() == kChunk ? harvest() : hipSuccess;
    };
    // the launch sequence of gsn_step(nsteps)
    for (const Launch &L : g->entry) HIP_TRY(timed(L));
    for (const Launch &L : g->kin_half) HIP_TRY(timed(L));
    for (int64_t i = 0; i < nsteps; ++i) {
        for (const Launch &L : g->nonlin) HIP_TRY(timed(L));
        for (const Launch &L : (i + 1 < nsteps ? g->kin_full : g->kin_half)) HIP_TRY(timed(L));
    }
    for (const Launch &L : g->exit_) HIP_TRY(timed(L));
    HIP_TRY(harvest());
    for (int i = 0; i < P_COUNT; ++i) ms[i] = cnt[i] ? tot[i] / cnt[i] : 0.0;
    return gsn_sync(g);
}

// ------------------------------------------------------------------ schedule autotuning
static_assert(kSmallVariant == kNumVariants - 1, "the autotuner leaves s4 out as the last variant");
// Largest grid that the autotuner tries s4 on: at 2^20 points it still wins
// the x passes of some shapes, at 2^22 none (twice the LDS per point).
constexpr long long kSmallPoints = 1LL << 21;

extern "C" int gsn_variant_count(void) { return kNumVariants; }

extern "C" const char *gsn_variant_name(int v)
{
    return (v >= 0 && v < kNumVariants) ? kVariantNames[v] : "";
}

extern "C" gsn_status gsn_get_schedule(gsn_grid g, int *variants, int npass)
{
    if (!g || !variants || npass < P_COUNT) return fail(GSN_EINVAL, "bad schedule arguments");
    for (int i = 0; i < P_COUNT; ++i) variants[i] = g->var[i];
    return GSN_OK;
}

extern "C" gsn_status gsn_set_schedule(gsn_grid g, const int *variants, int npass)
{
    if (!g || !variants || npass < P_COUNT) return fail(GSN_EINVAL, "bad schedule arguments");
    for (int i = 0; i < P_COUNT; ++i)
        if (variants[i] < 0 || variants[i] >= kNumVariants) return fail(GSN_EINVAL, "unknown schedule variant");
    HIP_TRY(hipSetDevice(g->device));
    HIP_TRY(hipStreamSynchronize(g->stream));
    for (int i = 0; i < P_COUNT; ++i) g->var[i] = variants[i];
    build_schedule(g);
    return GSN_OK;
}

// Launches that may follow each other in place on the data of one fill.
constexpr int kTimedLaunches = 8;

// The launch of pass p in the current step schedule, redirected from psi to the
// scratch buffer and with the end-of-step reduction switched off, so timing it
// leaves the solver state untouched.  What it runs is what the step runs; only the
// factors of values are chosen so that kTimedLaunches in place keep data in range:
// the entry and exit transforms are unitary, the kernel and the Laplacians are 1 / N
// in the middle of the spectrum (on a step's own factor, 1 / (2 P), complex64
// underflows within a few launches).  The plain y transforms keep their scale of 1,
// which spares them two multiplications a point; they grow the norm by sqrt(Ny).
static bool timing_launch(gsn_grid g, int p, Launch *out)
{
    const std::vector<Launch> *lists[] = {&g->entry, &g->kin_full, &g->nonlin, &g->exit_};
    for (const std::vector<Launch> *lst : lists)
        for (const Launch &L : *lst)
            if (L.pass == p) {
                *out = L;
                if (out->em) {
                    if (out->ea.psi == g->psi) out->ea.psi = g->scratch;
                } else {
                    if (out->la.s0.ptr == g->psi) out->la.s0.ptr = g->scratch;
                    out->la.reduce = 0;
                }
                if (p == P_ENTRY || p == P_EXIT) out->ea.scale = 1.0 / std::sqrt((double)g->Nx);
                if (p == P_KERNEL || p == P_LAPLACIAN || p == P_LAP_RHO) {
                    double lo = 1e300, hi = 0.0;
                    for (int d = 0; d < g->ndim; ++d) {
                        const double k1 = wavenumber(1, g->n[d], g->L[d]), kn = wavenumber(g->n[d] / 2, g->n[d], g->L[d]);
                        lo = std::min(lo, k1 * k1);
                        hi += kn * kn;
                    }
                    const double k2 = std::sqrt(lo * hi);
                    const double N = g->ndim == 3 ? g->Nz : g->Ny;
                    LmArgs &a = out->la;
                    const double mid = p == P_KERNEL ? std::fabs(a.cN / k2 + a.cY / (k2 + a.mY2) + a.c0) : k2 * a.scale;
                    const double f = 1.0 / (N * mid);
                    if (std::isfinite(f) && f > 0.0) {   // otherwise no kernel, or a pole
                        a.cN *= f;
                        a.cY *= f;
                        a.c0 *= f;
                        a.scale *= f;
                    }
                }
                return true;
            }
    return false;
}

// The data pass p is timed on: a copy of psi in scratch and, behind the density
// pass, the half spectra that pass makes of it.
static gsn_status timing_fill(gsn_grid g, int p)
{
    if (g->have_psi)
        HIP_TRY(hipMemcpyAsync(g->scratch, g->psi, g->esz * g->P, hipMemcpyDeviceToDevice, g->stream));
    Launch L;
    if (p > P_DENSITY && p != P_EXIT && timing_launch(g, P_DENSITY, &L)) HIP_TRY(launch(L, g->stream));
    return GSN_OK;
}

// Average of iters launches of pass p on fresh data: filled again, and two launches
// left out, every kTimedLaunches.
static gsn_status time_launch(gsn_grid g, int p, const Launch &L, int iters, double *ms)
{
    constexpr int kUntimed = 2;
    hipEvent_t a, b;
    HIP_TRY(hipEventCreate(&a));
    HIP_TRY(hipEventCreate(&b));
    double total = 0.0;
    for (int done = 0; done < iters;) {
        const int n = std::min(iters - done, kTimedLaunches - kUntimed);
        const gsn_status s = timing_fill(g, p);
        if (s) return s;
        for (int i = 0; i < kUntimed; ++i) HIP_TRY(launch(L, g->stream));
        HIP_TRY(hipEventRecord(a, g->stream));
        for (int i = 0; i < n; ++i) HIP_TRY(launch(L, g->stream));
        HIP_TRY(hipEventRecord(b, g->stream));
        HIP_TRY(hipEventSynchronize(b));
        float t = 0.f;
        HIP_TRY(hipEventElapsedTime(&t, a, b));
        total += t;
        done += n;
    }
    HIP_TRY(hipEventDestroy(a));
    HIP_TRY(hipEventDestroy(b));
    *ms = total / iters;
    return GSN_OK;
}

// Time a whole merged step (the kinetic passes, then the nonlinear sub-step
// density .. phase) on the scratch buffer.  The nonlinear mode changes what
// the x passes leave in the caches for the strided passes around them, so the
// sub-step timed alone can rank the modes the wrong way round (at 512^3 it
// preferred mode 0, whose whole steps were 1.6% slower).
static gsn_status time_nonlinear(gsn_grid g, int iters, double *ms)
{
    std::vector<Launch> seq;
    std::vector<Launch> step(g->kin_full);
    step.insert(step.end(), g->nonlin.begin(), g->nonlin.end());
    for (const Launch &L0 : step) {
        Launch L = L0;
        if (L.em) {
            if (L.ea.psi == g->psi) L.ea.psi = g->scratch;
        } else {
            if (L.la.s0.ptr == g->psi) L.la.s0.ptr = g->scratch;
            L.la.reduce = 0;
        }
        seq.push_back(L);
    }
    hipEvent_t a, b;
    HIP_TRY(hipEventCreate(&a));
    HIP_TRY(hipEventCreate(&b));
    for (const Launch &L : seq) HIP_TRY(launch(L, g->stream));
    HIP_TRY(hipEventRecord(a, g->stream));
    for (int i = 0; i < iters; ++i)
        for (const Launch &L : seq) HIP_TRY(launch(L, g->stream));
    HIP_TRY(hipEventRecord(b, g->stream));
    HIP_TRY(hipEventSynchronize(b));
    float t = 0.f;
    HIP_TRY(hipEventElapsedTime(&t, a, b));
    HIP_TRY(hipEventDestroy(a));
    HIP_TRY(hipEventDestroy(b));
    *ms = (double)t / iters;
    return GSN_OK;
}

static std::string cache_key(gsn_grid g, int p)
{
    hipDeviceProp_t prop;
    std::string arch = "unknown";
    if (hipGetDeviceProperties(&prop, g->device) == hipSuccess) arch = prop.gcnArchName;
    const size_t colon = arch.find(':');
    if (colon != std::string::npos) arch = arch.substr(0, colon);
    std::ostringstream k;
    k << arch << " " << g->ndim << "d";
    for (int d = 0; d < g->ndim; ++d) k << (d ? "x" : " ") << g->n[d];
    k << " " << (p < P_COUNT ? kPassNames[p] : "nonlinear_mode");
    if (g->storage == GSN_C128) k << "+c128";
    if (g->local_on) k << (g->bohm_on ? "+eq15b" : "+eq15");
    if (g->fld_gamma || g->fld_beta || g->fld_V) k << "+fields";
    return k.str();
}

static std::map<std::string, int> read_cache(const char *path)
{
    std::map<std::string, int> m;
    std::ifstream f(path);
    std::string line;
    while (std::getline(f, line)) {
        const size_t sp = line.rfind(' ');
        if (sp == std::string::npos) continue;
        const int v = std::atoi(line.c_str() + sp + 1);
        if (v >= 0 && v < kNumVariants) m[line.substr(0, sp)] = v;
    }
    return m;
}

extern "C" gsn_status gsn_autotune(gsn_grid g, int iters)
{
    if (!g) return fail(GSN_EINVAL, "grid is NULL");
    if (iters < 1 || iters > 10000) return fail(GSN_EINVAL, "iters must be in [1, 10000]");
    HIP_TRY(hipSetDevice(g->device));
    // realistic data for timing: a copy of psi (or zeros before psi is set)
    if (g->have_psi)
        HIP_TRY(hipMemcpyAsync(g->scratch, g->psi, g->esz * g->P, hipMemcpyDeviceToDevice, g->stream));
    else
        HIP_TRY(hipMemsetAsync(g->scratch, 0, g->esz * g->P, g->stream));
    const char *cpath = std::getenv("GSN_AUTOTUNE_CACHE");
    std::map<std::string, int> cache;
    if (cpath && *cpath) cache = read_cache(cpath);
    std::vector<std::string> fresh;
    // the latency form is no candidate for grids that fill the chip
    const int nvar = g->P > kSmallPoints ? kSmallVariant : kNumVariants;
    bool present[P_COUNT] = {};   // passes this grid's step has
    int from_file = 0;
    g->store_psi = 0;
    for (int p = 0; p < P_COUNT; ++p) {
        const std::string key = cache_key(g, p);
        auto it = cache.find(key);
        if (it != cache.end()) {
            g->var[p] = it->second;
            ++from_file;
            continue;
        }
        int best = g->var[p];
        double best_ms = 1e300;
        for (int v = 0; v < nvar; ++v) {
            g->var[p] = v;
            build_schedule(g);
            Launch L;
            if (!timing_launch(g, p, &L)) break;
            present[p] = true;
            double ms = 0.0;
            gsn_status s = time_launch(g, p, L, iters, &ms);
            if (s) return s;
            if (ms < best_ms) { best_ms = ms; best = v; }
        }
        g->var[p] = best;
        if (present[p]) fresh.push_back(key + " " + std::to_string(best));
    }
    // nonlinear sub-step: recompute psi in the phase pass (mode 0), or store
    // real-space psi in the density pass (mode 1, with its own variants of the
    // two x passes); whole steps are timed because the two passes change
    // together and change the strided passes' cache state
    const std::string mkey = cache_key(g, P_COUNT);
    auto mit = cache.find(mkey);
    if (mit != cache.end()) {
        g->store_psi = mit->second ? 1 : 0;
    } else {
        build_schedule(g);
        double best_ms = 0.0;
        gsn_status s = time_nonlinear(g, iters, &best_ms);
        if (s) return s;
        // mode 1: the density pass's variant with the phase pass as it is,
        // then the phase pass's with the best of those (every pair of the two
        // would take 36 timings for the same choice)
        const int d0 = g->var[P_DENSITY], h0 = g->var[P_PHASE];
        int bd = d0, bh = h0, bm = 0;
        double mode1_ms = 1e300;
        g->store_psi = 1;
        for (int pass : {P_DENSITY, P_PHASE})
            for (int v = 0; v < nvar; ++v) {
                const int vd = pass == P_DENSITY ? v : bd, vh = pass == P_DENSITY ? h0 : v;
                if (pass == P_PHASE && v == h0) continue;   // timed already
                g->var[P_DENSITY] = vd;
                g->var[P_PHASE] = vh;
                build_schedule(g);
                double ms = 0.0;
                if ((s = time_nonlinear(g, iters, &ms))) return s;
                if (ms < mode1_ms) { mode1_ms = ms; bd = vd; bh = vh; }
            }
        bm = mode1_ms < best_ms;
        g->store_psi = bm;
        g->var[P_DENSITY] = bm ? bd : d0;
        g->var[P_PHASE] = bm ? bh : h0;
        if (bm) {
            fresh.push_back(cache_key(g, P_DENSITY) + " " + std::to_string(g->var[P_DENSITY]));
            fresh.push_back(cache_key(g, P_PHASE) + " " + std::to_string(g->var[P_PHASE]));
        }
        // s4 throughout, by whole steps: on small grids the passes differ by
        // less than the noise of timing them one by one
        double chosen_ms = bm ? mode1_ms : best_ms;
        if (nvar == kNumVariants && from_file == 0) {
            int keep[P_COUNT];
            std::copy(g->var, g->var + P_COUNT, keep);
            for (int p = 0; p < P_COUNT; ++p)
                if (p != P_ENTRY && p != P_EXIT && present[p]) g->var[p] = kSmallVariant;
            int mode = -1;
            for (int m = 0; m < 2; ++m) {
                g->store_psi = m;
                build_schedule(g);
                double ms = 0.0;
                if ((s = time_nonlinear(g, iters, &ms))) return s;
                if (ms < chosen_ms) { chosen_ms = ms; mode = m; }
            }
            g->store_psi = mode < 0 ? bm : mode;
            if (mode < 0) std::copy(keep, keep + P_COUNT, g->var);
            else
                for (int p = 0; p < P_COUNT; ++p)
                    if (g->var[p] != keep[p]) fresh.push_back(cache_key(g, p) + " " + std::to_string(g->var[p]));
        }
        fresh.push_back(mkey + " " + std::to_string(g->store_psi));
    }
    build_schedule(g);
    if (cpath && *cpath && !fresh.empty()) {
        std::ofstream f(cpath, std::ios::app);
        for (const std::string &l : fresh) f << l << "\n";
    }
    return GSN_OK;
}

extern "C" gsn_status gsn_set_nonlinear_mode(gsn_grid g, int mode)
{
    if (!g) return fail(GSN_EINVAL, "grid is NULL");
    if (mode != 0 && mode != 1) return fail(GSN_EINVAL, "mode must be 0 or 1");
    HIP_TRY(hipSetDevice(g->device));
    HIP_TRY(hipStreamSynchronize(g->stream));
    g->store_psi = mode;
    build_schedule(g);
    return GSN_OK;
}

extern "C" gsn_status gsn_get_nonlinear_mode(gsn_grid g, int *mode)
{
    if (!g || !mode) return fail(GSN_EINVAL, "NULL argument");
    *mode = g->store_psi;
    return GSN_OK;
}

// ------------------------------------------------------------------ coarse steps and the learned corrector
extern "C" gsn_status gsn_set_coarse_ratio(gsn_grid g, int ratio)
{
    if (!g) return fail(GSN_EINVAL, "grid is NULL");
    if (ratio < 0 || ratio > 4096) return fail(GSN_EINVAL, "ratio must be in [0, 4096]");
    if (ratio > 0 && !g->have_dz) return fail(GSN_ESTATE, "set the coefficients (dz) first");
    HIP_TRY(hipSetDevice(g->device));
    HIP_TRY(hipStreamSynchronize(g->stream));
    g->coarse_ratio = ratio;
    gsn_status s = upload_kinetic(g);
    if (s) return s;
    build_schedule(g);
    return GSN_OK;
}

static gsn_status run_potential(gsn_grid g, float *dst)
{
    for (Launch L : g->pot) {
        if (L.em) L.ea.phi = dst;
        HIP_TRY(launch(L, g->stream));
    }
    return GSN_OK;
}

extern "C" gsn_status gsn_potential(gsn_grid g, float *phi_dev)
{
    if (!g || !phi_dev) return fail(GSN_EINVAL, "NULL argument");
    if (g->fld_gamma || g->fld_beta) return fail(GSN_EUNSUPPORTED, "no potential readout with source fields");
    if (g->storage == GSN_C128) return fail(GSN_EUNSUPPORTED, "no potential readout on FP64-storage grids");
    if (!g->have_psi) return fail(GSN_ESTATE, "psi not set");
    HIP_TRY(hipSetDevice(g->device));
    return run_potential(g, phi_dev);
}

static gsn_status run_lists(gsn_grid g, const StepLists &L, int64_t nsteps)
{
    gsn_status s;
    if ((s = run_list(g, L.entry)) || (s = run_list(g, L.kin_half))) return s;
    for (int64_t i = 0; i < nsteps; ++i) {
        if ((s = run_list(g, L.nonlin))) return s;
        if ((s = run_list(g, i + 1 < nsteps ? L.kin_full : L.kin_half))) return s;
    }
    return run_list(g, L.exit_);
}

extern "C" gsn_status gsn_step_coarse(gsn_grid g, int64_t nsteps)
{
    gsn_status s = ready(g);
    if (s) return s;
    if (g->coarse_ratio <= 0) return fail(GSN_ESTATE, "no coarse ratio set");
    if (nsteps < 0) return fail(GSN_EINVAL, "nsteps must be >= 0");
    if (nsteps == 0) return GSN_OK;
    HIP_TRY(hipSetDevice(g->device));
    return run_lists(g, g->coarse, nsteps);
}

extern "C" gsn_status gsn_step_corrected(gsn_grid g, gsn_corrector c, int64_t ncoarse, int audit_every, double tol,
                                         int64_t *n_fallbacks, double *max_audit_err)
{
    gsn_status s = ready(g);
    if (s) return s;
    if (!c) return fail(GSN_EINVAL, "corrector is NULL");
    if (g->ndim != 2) return fail(GSN_EUNSUPPORTED, "the corrector works on 2-D grids");
    if (g->fld_gamma || g->fld_beta) return fail(GSN_EUNSUPPORTED, "no corrected steps with source fields");
    if (g->storage == GSN_C128) return fail(GSN_EUNSUPPORTED, "the corrector works on complex64 grids");
    if (corrector_height(c) != g->n[0] || corrector_width(c) != g->n[1])
        return fail(GSN_EINVAL, "corrector image size differs from the grid");
    if (g->coarse_ratio <= 0) return fail(GSN_ESTATE, "no coarse ratio set");
    if (ncoarse < 0 || audit_every < 0 || !(tol >= 0.0)) return fail(GSN_EINVAL, "bad stepping arguments");
    HIP_TRY(hipSetDevice(g->device));
    int64_t nfb = 0;
    double worst = 0.0;
    float *phi = corrector_phi_buffer(c);
    float2 *saved = corrector_psi_buffer(c, 0), *corrected = corrector_psi_buffer(c, 1);
    const size_t bytes = 8ull * g->P;
    for (int64_t i = 0; i < ncoarse; ++i) {
        const bool audit = audit_every > 0 && ((i + 1) % audit_every == 0);
        if (audit) {
            HIP_TRY(hipMemcpyAsync(saved, g->psi, bytes, hipMemcpyDeviceToDevice, g->stream));
            HIP_TRY(hipMemcpyAsync(g->st_save[0], g->st, sizeof(DevState), hipMemcpyDeviceToDevice, g->stream));
        }
        float2 *const spare = corrector_fused(c) ? corrector_spare(c) : nullptr;
        const float2 *coarse = g->psi;   // the coarse step's state
        if (!g->pot_spec.empty()) {
            // one coarse step without its closing inverse x transform, which
            // the readout's first pass performs while it forms the density; for
            // the fused network it leaves psi in the spare image, so that the
            // network can write the state back where it belongs (a copy of the
            // state less per coarse step: 512^2 5 of 90 us)
            const StepLists &C = g->coarse;
            if ((s = run_list(g, C.entry)) || (s = run_list(g, C.kin_half)) || (s = run_list(g, C.nonlin)) ||
                (s = run_list(g, C.kin_half)))
                return s;
            for (Launch L : g->pot_spec) {
                if (L.em) L.ea.phi = phi;
                if (L.pass == P_DENSITY && spare) L.ea.psi_st = spare;
                HIP_TRY(launch(L, g->stream));
            }
            if (spare) coarse = spare;
        } else {
            if ((s = run_lists(g, g->coarse, 1))) return s;
            if ((s = run_potential(g, phi))) return s;
        }
        if ((s = corrector_correct(c, coarse, phi, g->psi, &g->st->theta, g->stream))) {
            // without the network's result the coarse step's state is the state
            if (coarse != g->psi)
                (void)hipMemcpyAsync(g->psi, coarse, bytes, hipMemcpyDeviceToDevice, g->stream);
            return s;
        }
        if (audit) {
            // the fine solver from the same state is the reference for the corrected step
            HIP_TRY(hipMemcpyAsync(corrected, g->psi, bytes, hipMemcpyDeviceToDevice, g->stream));
            HIP_TRY(hipMemcpyAsync(g->st_save[1], g->st, sizeof(DevState), hipMemcpyDeviceToDevice, g->stream));
            HIP_TRY(hipMemcpyAsync(g->psi, saved, bytes, hipMemcpyDeviceToDevice, g->stream));
            HIP_TRY(hipMemcpyAsync(g->st, g->st_save[0], sizeof(DevState), hipMemcpyDeviceToDevice, g->stream));
            StepLists fine{g->entry, g->kin_half, g->kin_full, g->nonlin, g->exit_};
            if ((s = run_lists(g, fine, g->coarse_ratio))) return s;
            const int nb = 256;
            hipLaunchKernelGGL(k_state_diff, dim3(nb), dim3(256), 0, g->stream, corrected, g->st_save[1], g->psi,
                               g->st, g->P, g->epart);
            HIP_TRY(hipGetLastError());
            std::vector<double> h(2 * nb);
            HIP_TRY(hipMemcpyAsync(h.data(), g->epart, 16ull * nb, hipMemcpyDeviceToHost, g->stream));
            HIP_TRY(hipStreamSynchronize(g->stream));
            double d = 0.0, n = 0.0;
            for (int b = 0; b < nb; ++b) { d += h[2 * b]; n += h[2 * b + 1]; }
            const double err = n > 0.0 ? std::sqrt(d / n) : 0.0;
            if (!(err <= worst)) worst = err;
            if (!(err <= tol)) {
                ++nfb;   // keep the fine result already in psi
            } else {
                HIP_TRY(hipMemcpyAsync(g->psi, corrected, bytes, hipMemcpyDeviceToDevice, g->stream));
                HIP_TRY(hipMemcpyAsync(g->st, g->st_save[1], sizeof(DevState), hipMemcpyDeviceToDevice, g->stream));
            }
        }
    }
    if (n_fallbacks) *n_fallbacks = nfb;
    if (max_audit_err) *max_audit_err = worst;
    return GSN_OK;
}
