// gsn_batch.hip -- many independent 2-D instances (uneven sizes, per-instance
// kernel and coefficients) advanced together.
//
// Instances with the same shape form a group.  Every pass of a group is ONE
// grouped launch: block b works on tile (b mod tpi) of instance (b / tpi),
// whose arguments (buffers, tables, coefficients) sit in a device array, so a
// pass over 20 instances of 1024^2 is a single launch of thousands of blocks.
// Groups only depend on themselves, so gsn_batch_step captures each group's
// launch chain on its own stream branch of one hipGraph and replays the whole
// run with one hipGraphLaunch.  Mode 1 runs the same tiles from one persistent
// kernel that pulls (step, pass, instance, tile) work items from a device
// queue with per-instance completion counters.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <fstream>
#include <map>
#include <string>
#include <vector>

#include "gsn_host.hpp"
#include "gsn_queue.hpp"

namespace {

// ------------------------------------------------------------------ persistent kernel
// One 512-thread block shape serves every tile: x passes with 8 points per
// thread (EM), y passes with 16 (LM), so LINES = 512 * E / N.
constexpr int kPThreads = 512;
template <int N> struct PCfg {
    static constexpr int EE = 8, EL = kPThreads * EE / N;
    static constexpr int LE = 16, LL = kPThreads * LE / N;
};
constexpr int kPLds = 64 * 1024 / 8;   // float2 slots: max over the supported sizes

struct PInst {
    EmArgs em[Q_NKIND];
    LmArgs lm[Q_NKIND];
    int nx, ny;
};

// One queue per XCD: an instance's items all run on one XCD, whose L2 every
// CU of the XCD shares, so a tile hand-off needs only the producer's stores
// acknowledged (vmcnt 0) and the consumer's L1 invalidated - not an L2
// write-back and invalidate across XCDs, which made every hand-off cost more
// than the tile.
constexpr int kNQ = 8;
constexpr unsigned kQRun = 4;
struct PArgs {
    const PInst *inst;
    QTables T[kNQ];                 // queue x: its instances' tile prefixes
    const int *list[kNQ];           // queue x: local instance -> instance
    unsigned long long total[kNQ];  // queue x: items
    unsigned long long *head;       // kNQ counters
    unsigned long long *done;
    unsigned *err;
    unsigned spin_limit;
    int store_psi;
    unsigned long long fail_item;   // test hook: raise the error when this item is pulled (~0 = never)
};

template <int N> __device__ __noinline__ void p_em(int kind, const EmArgs &a, int tile, float2 *lds, double *sh,
                                                      int store)
{
    using C = PCfg<N>;
    if (kind == Q_ENTRY) em_fft_tile<N, C::EE, C::EL, -1>(a, tile, lds);
    else if (kind == Q_EXIT) em_fft_tile<N, C::EE, C::EL, 1>(a, tile, lds);
    else if (kind == Q_DENSITY) {
        if (store) density_tile<N, C::EE, C::EL, true>(a, tile, lds, sh);
        else density_tile<N, C::EE, C::EL, false>(a, tile, lds, sh);
    } else {
        if (store) phase_tile<N, C::EE, C::EL, false, true>(a, tile, lds, sh);
        else phase_tile<N, C::EE, C::EL, false, false>(a, tile, lds, sh);
    }
}

template <int N> __device__ __noinline__ void p_lm(int kind, const LmArgs &a, int tile, float2 *lds, double *sh)
{
    using C = PCfg<N>;
    if (kind == Q_KERNEL) lm_tile<N, C::LE, C::LL, LM_KERN>(a, tile, lds, sh);
    else lm_tile<N, C::LE, C::LL, LM_KIN>(a, tile, lds, sh);
}

__global__ void k_queue_reset(unsigned long long *head, unsigned long long *done, unsigned *err, int count)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < kNQ) head[i] = 0;
    if (i == 0) *err = 0;
    if (i < count) done[i] = 0;
}

// Blocks pull items of their XCD's queue in increasing order; an item waits
// (bounded) until its instance has completed every tile of the earlier phases.
// Exit: the queue is exhausted, or a wait exceeded spin_limit (then err is set
// and every block leaves at its next wait).  The host checks after the run
// that every non-empty queue was drained (a queue whose XCD ran no block).
__global__ __launch_bounds__(kPThreads) void k_batch_persistent(PArgs a)
{
    __shared__ float2 lds[kPLds];
    __shared__ double sh[kPThreads / 64 + 1];
    __shared__ unsigned long long s_item;
    __shared__ int s_stop, s_q;
    if (threadIdx.x == 0) s_q = (int)(__builtin_amdgcn_s_getreg(6164) & (kNQ - 1));   // HW_REG_XCC_ID
    __syncthreads();
    const int q = s_q;
    if (a.T[q].count == 0) return;
    const QTables &T = a.T[q];
    unsigned long long next = 0, end = 0;   // thread 0: this block's current run of items
    for (;;) {
        if (threadIdx.x == 0) {
            int stop = __hip_atomic_load(a.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
            unsigned long long x = 0;
            if (!stop) {
                // kQRun consecutive items per atomic on the queue head; a run
                // keeps the order (its items depend only on smaller numbers,
                // all handed out before it)
                if (next == end) {
                    next = atomicAdd(&a.head[q], (unsigned long long)kQRun);
                    end = next + kQRun;
                }
                x = next++;
                stop = x >= a.total[q];
                if (x == a.fail_item) {
                    atomicOr(a.err, 1u);
                    stop = 1;
                }
            }
            if (!stop) {
                const QItem it = qdecode(T, x);
                const int inst = a.list[q][it.inst];
                unsigned n = 0;
                while (__hip_atomic_load(&a.done[inst], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < it.need) {
                    if (++n > a.spin_limit || __hip_atomic_load(a.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
                        atomicOr(a.err, 1u);
                        stop = 1;
                        break;
                    }
                    __builtin_amdgcn_s_sleep(2);
                }
                // acquire: drop this CU's L1 copies, so the tiles the counter
                // covers are read from the shared L2 (sc1; with sc0, the
                // work-group scope, the L1 keeps its lines)
                asm volatile("buffer_inv sc1\n\ts_waitcnt vmcnt(0)" ::: "memory");
            }
            s_item = x;
            s_stop = stop;
        }
        __syncthreads();
        if (s_stop) break;
        const QItem it = qdecode(T, s_item);
        const int inst = a.list[q][it.inst];
        const PInst &I = a.inst[inst];
        const bool lm = it.kind == Q_KIN_HALF || it.kind == Q_KIN_FULL || it.kind == Q_KERNEL;
        if (lm) {
            switch (I.ny) {
            case 128: p_lm<128>(it.kind, I.lm[it.kind], it.tile, lds, sh); break;
            case 256: p_lm<256>(it.kind, I.lm[it.kind], it.tile, lds, sh); break;
            case 512: p_lm<512>(it.kind, I.lm[it.kind], it.tile, lds, sh); break;
            default: p_lm<1024>(it.kind, I.lm[it.kind], it.tile, lds, sh); break;
            }
        } else {
            switch (I.nx) {
            case 128: p_em<128>(it.kind, I.em[it.kind], it.tile, lds, sh, a.store_psi); break;
            case 256: p_em<256>(it.kind, I.em[it.kind], it.tile, lds, sh, a.store_psi); break;
            case 512: p_em<512>(it.kind, I.em[it.kind], it.tile, lds, sh, a.store_psi); break;
            default: p_em<1024>(it.kind, I.em[it.kind], it.tile, lds, sh, a.store_psi); break;
            }
        }
        // release within the XCD: this thread's stores acknowledged by the L2
        // before the block's count goes up
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (threadIdx.x == 0) atomicAdd(&a.done[inst], 1ull);
        __syncthreads();   // s_item / s_stop are rewritten next iteration
    }
}

bool persistent_size(int n) { return n == 128 || n == 256 || n == 512 || n == 1024; }


// ------------------------------------------------------------------ grouped kernel tables
// pipe: the density, phase, kinetic and kernel entries are the persistent
// prefetching kernels (arguments: array, tiles per instance, instances).
struct GKernels {
    int E, TPL, lm_lines, em_lines;
    bool pipe;
    const void *em_fwd, *em_inv;
    const void *density, *density_store, *phase, *phase_real;
    const void *lm_kin, *lm_kern;
    int lm_nt;   // threads of a strided block
    int lm_threads() const { return lm_nt; }
    int em_threads() const { return em_lines * TPL; }
};

template <int N, int V> GKernels make_gkernels()
{
    using C = Cfg<N, V>;
    constexpr int E = C::E, LL = C::LM_LINES, EL = C::EM_LINES;
    GKernels k;
    k.E = E;
    k.TPL = C::TPL;
    k.lm_lines = LL;
    k.lm_nt = LL * C::TPL;
    k.em_lines = EL;
    k.pipe = C::PIPE;
    k.em_fwd = (const void *)k_em_fft_g<N, E, EL, -1>;
    k.em_inv = (const void *)k_em_fft_g<N, E, EL, 1>;
    if constexpr (C::PIPE) {
        k.density = (const void *)k_densityp_g<N, E, EL, false>;
        k.density_store = (const void *)k_densityp_g<N, E, EL, true>;
        k.phase = (const void *)k_phasep_g<N, E, EL, false>;
        k.phase_real = (const void *)k_phasep_g<N, E, EL, true>;
        using T = TwoButterfly<N>;
        if constexpr (V == 3 && T::BATCH) {
            k.lm_kin = (const void *)k_lmp2_g<N, T::LINES, LM_KIN>;
            k.lm_kern = (const void *)k_lmp2_g<N, T::LINES, LM_KERN>;
            k.lm_lines = T::LINES;
            k.lm_nt = T::THREADS;
        } else {
            k.lm_kin = (const void *)k_lmp_g<N, E, LL, LM_KIN>;
            k.lm_kern = (const void *)k_lmp_g<N, E, LL, LM_KERN>;
        }
    } else {
        k.density = (const void *)k_density_g<N, E, EL, false>;
        k.density_store = (const void *)k_density_g<N, E, EL, true>;
        k.phase = (const void *)k_phase_g<N, E, EL, false>;
        k.phase_real = (const void *)k_phase_g<N, E, EL, true>;
        k.lm_kin = (const void *)k_lm_g<N, E, LL, LM_KIN>;
        k.lm_kern = (const void *)k_lm_g<N, E, LL, LM_KERN>;
    }
    return k;
}

template <int N> const GKernels *gvariant(int v)
{
    static const GKernels k[kNumBatchVariants] = {make_gkernels<N, 0>(), make_gkernels<N, 1>(), make_gkernels<N, 2>(),
                                                  make_gkernels<N, 3>()};
    return &k[v];
}

const GKernels *gkernels_for(int N, int v)
{
    if (v < 0 || v >= kNumBatchVariants) v = 0;
    switch (N) {
    case 8: return gvariant<8>(v);
    case 16: return gvariant<16>(v);
    case 32: return gvariant<32>(v);
    case 64: return gvariant<64>(v);
    case 128: return gvariant<128>(v);
    case 256: return gvariant<256>(v);
    case 512: return gvariant<512>(v);
    case 1024: return gvariant<1024>(v);
    case 2048: return gvariant<2048>(v);
    default: return nullptr;
    }
}

// pass kinds of a 2-D step
enum BKind { B_ENTRY = 0, B_KIN_HALF, B_KIN_FULL, B_DENSITY, B_KERNEL, B_PHASE, B_EXIT, B_NKIND };
// schedule variant per pass family: kinetic, density, kernel, phase, entry/exit
enum BFam { F_KIN = 0, F_DENSITY, F_KERNEL, F_PHASE, F_XFFT, F_NFAM };
const int kFamOf[B_NKIND] = {F_XFFT, F_KIN, F_KIN, F_DENSITY, F_KERNEL, F_PHASE, F_XFFT};

struct Instance {
    int ny, nx;
    double Ly, Lx;
    long long P;
    float2 *psi, *half, *nyq;
    double *mass_parts;
    DevState *st;
    double2 *tw_x, *tw_y, *kinF_x, *kinF_y, *kinH_x, *kinH_y;
    double *k2_x, *k2_y;
    gsn_kernel kern;
    double a, g, dz;
    bool set;
};

struct GLaunch {
    const void *fn;
    dim3 grid, block;
    const void *args;   // device array of EmArgs or LmArgs
    int tpi;
    int count;          // instances (persistent kernels walk count * tpi tiles)
    bool pipe;
    bool operator==(const GLaunch &o) const
    {
        return fn == o.fn && grid.x == o.grid.x && block.x == o.block.x && args == o.args && tpi == o.tpi &&
               count == o.count && pipe == o.pipe;   // one-dimensional launches
    }
};

struct Group {
    int ny, nx;
    std::vector<int> members;
    // schedule of this shape group: variant per pass family, nonlinear mode
    // (1: the density pass stores real-space psi); set for every group by
    // gsn_batch_set_schedule, per group by gsn_batch_autotune
    int var[F_NFAM];
    int store_psi;
    GLaunch launch[B_NKIND];
    void *args_dev[B_NKIND];   // device arrays (inside the workspace)
};

}  // namespace

struct gsn_batch_ {
    int count;
    hipStream_t user;     // the caller's stream (may be the NULL stream)
    hipStream_t stream;   // internal stream: capture, replay, copies
    hipEvent_t ev_in, ev_out;
    int device;
    std::vector<Instance> inst;
    std::vector<Group> groups;
    std::vector<hipStream_t> side;   // one capture branch per group
    int var[F_NFAM];
    int store_psi;
    int mode;   // 0 grouped launches in a graph, 1 persistent kernel
    char *ws;
    size_t ws_bytes;
    float2 *scratch;   // readout staging, 16 * max P bytes or more
    size_t scratch_bytes;
    char *st;          // the instances' states
    double *k2_unit;
    double2 *kin_unit;
    double2 *sct;      // sin / cos table of the persistent phase pass
    // graph cache
    hipGraphExec_t exec;
    int64_t exec_steps;
    bool dirty;
    // persistent mode state (inside the workspace)
    void *pq;
    unsigned long long *q_head, *q_done;
    unsigned *q_err, *q_prefix;
    PInst *q_inst;
    std::vector<unsigned> h_prefix;   // per queue: tile prefixes, then (at list_off) its instances
    int q_count[kNQ], q_pre_off[kNQ], q_list_off[kNQ];
    unsigned long long q_total[kNQ];   // items of the last run, per queue
    bool q_built;
    unsigned spin_limit;
    long long fail_item;
};

namespace {

const int kMaxInstances = 4096;

struct BLayout {
    std::vector<size_t> inst_off;
    size_t args_off, scratch_off, scratch_bytes, unit_off, queue_off, st_off, total;
};

// The instances' states lie in one array, a stride apart (no two share a cache
// line: different XCDs write them), so that one copy reads them all.
constexpr size_t kStateStride = 256;
static_assert(sizeof(DevState) <= kStateStride, "state stride");
// values of the mass partials of one instance, as the read-out takes them
constexpr int kMassParts = 256;

// bytes of one instance's region (buffers, partials, tables)
size_t instance_bytes(int ny, int nx)
{
    const long long P = (long long)ny * nx;
    int db = 0;
    for (int v = 0; v < kNumVariants; ++v) {
        const NKernels *k = kernels_for(nx, v);
        db = std::max(db, (int)((ny / 2 + k->em_lines - 1) / k->em_lines));
    }
    size_t b = 0;
    b += align256(8ull * P);                 // psi
    b += align256(4ull * P);                 // half spectrum
    b += align256(8ull * ny);                // Nyquist column
    b += align256(8ull * db);                // mass partials
    b += 6 * align256(16ull * std::max(nx, ny));   // twiddles and kinetic factors
    b += 2 * align256(8ull * std::max(nx, ny));    // |k|^2 tables
    return b;
}

gsn_status compute_blayout(int count, const int32_t *n, BLayout *L)
{
    size_t off = 0;
    long long maxP = 0;
    L->inst_off.resize(count);
    for (int i = 0; i < count; ++i) {
        L->inst_off[i] = off;
        off += instance_bytes(n[2 * i], n[2 * i + 1]);
        maxP = std::max(maxP, (long long)n[2 * i] * n[2 * i + 1]);
    }
    L->args_off = off;
    off += align256((size_t)B_NKIND * count * std::max(sizeof(EmArgs), sizeof(LmArgs)));
    L->scratch_off = off;
    L->scratch_bytes = align256(std::max(16ull * maxP, 8ull * kMassParts * std::min(count, 64)));
    off += L->scratch_bytes;
    L->unit_off = off;
    off += 512 + 16 * kSinCosTable;
    L->queue_off = off;
    off += align256(256) + align256(8ull * count) + align256(4ull * (Q_NKIND * (count + kNQ) + count)) +
           align256(sizeof(PInst) * (size_t)count);
    L->st_off = off;
    off += kStateStride * count;
    L->total = off;
    return GSN_OK;
}

gsn_status validate_batch(int count, int ndim, const int32_t *n)
{
    if (count < 1 || count > kMaxInstances) return fail(GSN_EINVAL, "count must be in [1, 4096]");
    if (ndim != 2) return fail(GSN_EUNSUPPORTED, "batched instances are 2-D");
    if (!n) return fail(GSN_EINVAL, "n is NULL");
    for (int i = 0; i < 2 * count; ++i)
        if (!is_pow2(n[i]) || n[i] < 8 || n[i] > 2048)
            return fail(GSN_EUNSUPPORTED, "every extent must be a power of two in [8, 2048]");
    return GSN_OK;
}

gsn_status upload_sync(hipStream_t s, void *dst, const void *src, size_t bytes)
{
    HIP_TRY(hipMemcpyAsync(dst, src, bytes, hipMemcpyHostToDevice, s));
    HIP_TRY(hipStreamSynchronize(s));
    return GSN_OK;
}

// An instance's tables lie one after the other (tw_x first, k2_y last): filled in
// a host copy, uploaded in one transfer.
gsn_status upload_instance_tables(gsn_batch b, Instance &I)
{
    const int dims[2] = {I.nx, I.ny};
    const double Ls[2] = {I.Lx, I.Ly};
    double2 *tw[2] = {I.tw_x, I.tw_y}, *kf[2] = {I.kinF_x, I.kinF_y}, *kh[2] = {I.kinH_x, I.kinH_y};
    double *k2[2] = {I.k2_x, I.k2_y};
    std::vector<char> host((char *)(I.k2_y + I.ny) - (char *)I.tw_x);
    auto at = [&](void *dev) { return host.data() + ((char *)dev - (char *)I.tw_x); };
    for (int d = 0; d < 2; ++d) {
        const int N = dims[d];
        double2 *t = (double2 *)at(tw[d]), *f = (double2 *)at(kf[d]), *h = (double2 *)at(kh[d]);
        double *q = (double *)at(k2[d]);
        for (int j = 0; j < N; ++j) {
            const double ang = 2.0 * M_PI * (double)j / (double)N;
            t[j] = make_double2(std::cos(ang), -std::sin(ang));
            const double k = wavenumber(j, N, Ls[d]);
            q[j] = k * k;
            const double thf = -I.a * k * k * I.dz, thh = 0.5 * thf;
            f[j] = make_double2(std::cos(thf), std::sin(thf));
            h[j] = make_double2(std::cos(thh), std::sin(thh));
        }
    }
    return upload_sync(b->stream, I.tw_x, host.data(), host.size());
}

double kernel_k0(const gsn_kernel &k)
{
    double v = k.c_contact;
    if (k.c_yukawa != 0.0) v += k.c_yukawa / (k.m_yukawa * k.m_yukawa);
    return v;
}

// Per-instance argument structs of one pass kind (same layout as one grid).
EmArgs em_args(gsn_batch b, const Instance &I, int kind)
{
    EmArgs a;
    std::memset(&a, 0, sizeof(a));
    a.psi = I.psi;
    a.half = I.half;
    a.nyq = I.nyq;
    a.tw = I.tw_x;
    a.sct = b->sct;
    a.scale = kind == B_EXIT ? 1.0 / I.nx : 1.0;
    a.g = I.g;
    a.dz = I.dz;
    a.partials = I.mass_parts;
    a.nlines = (kind == B_ENTRY || kind == B_EXIT) ? I.ny : I.ny / 2;
    return a;
}

Seg seg_of(float2 *ptr, long long es, long long ls, long long os, int nlines, int nouter, int lpt)
{
    Seg s;
    std::memset(&s, 0, sizeof(s));
    s.ptr = ptr;
    s.es = es;
    s.ls = ls;
    s.os = os;
    s.nlines = nlines;
    s.ngroups = (nlines + lpt - 1) / lpt;
    s.ntiles = s.ngroups * nouter;
    return s;
}

LmArgs lm_args(gsn_batch b, const Instance &I, int kind, int lpt, int var_density)
{
    LmArgs a;
    std::memset(&a, 0, sizeof(a));
    a.kin1 = a.kin2 = a.kinp = b->kin_unit;
    a.k2_1 = a.k2_2 = a.k2_p = b->k2_unit;
    a.st = I.st;
    a.tw = I.tw_y;
    const int H = I.nx / 2;
    if (kind == B_KIN_HALF || kind == B_KIN_FULL) {
        a.scale = 1.0 / I.ny;
        a.s0 = seg_of(I.psi, I.nx, 1, 0, I.nx, 1, lpt);
        a.s0.c1l = 1;
        a.kin1 = kind == B_KIN_HALF ? I.kinH_x : I.kinF_x;
        a.kinp = kind == B_KIN_HALF ? I.kinH_y : I.kinF_y;
    } else {   // B_KERNEL
        // the scale from rho to phi, with the split's 1/2 (as for one grid)
        const double sk = 0.5 / (double)I.P;
        a.scale = 1.0;
        a.s0 = seg_of(I.half, H, 1, 0, H, 1, lpt);
        a.s0.c1l = 1;
        a.s1 = seg_of(I.nyq, 1, 0, 0, 1, 1, lpt);
        a.s1.c1f = H;
        a.k2_1 = I.k2_x;
        a.k2_p = I.k2_y;
        a.cN = I.kern.c_newton * sk;
        a.cY = I.kern.c_yukawa * sk;
        a.mY2 = I.kern.m_yukawa * I.kern.m_yukawa;
        a.c0 = I.kern.c_contact * sk;
        a.reduce = 1;
        a.mass_parts = I.mass_parts;
        const NKernels *kx = kernels_for(I.nx, var_density);
        a.nmass = (I.ny / 2 + kx->em_lines - 1) / kx->em_lines;
        a.k0_dz_over_P = kernel_k0(I.kern) * I.dz / (double)I.P;
    }
    return a;
}

// The persistent grouped kernels keep the first instance's tables (twiddles,
// kinetic factors, |k|^2) in LDS for every instance of the group: only valid
// when every member would have built identical tables.
bool same_tables(gsn_batch b, const Group &G)
{
    const Instance &I0 = b->inst[G.members[0]];
    for (int m : G.members) {
        const Instance &I = b->inst[m];
        if (I.Lx != I0.Lx || I.Ly != I0.Ly || I.a != I0.a || I.dz != I0.dz) return false;
    }
    return true;
}

// Rebuild one group's launch descriptors and upload its argument arrays (which lie
// one after the other) in one transfer.  The recorded graph reads the arguments
// from there, so it stays while the launches do.
constexpr size_t kArgBytes = std::max(sizeof(EmArgs), sizeof(LmArgs));
gsn_status build_group(gsn_batch b, Group &G)
{
    const int cnt = (int)G.members.size();
    const bool uniform = same_tables(b, G);
    std::vector<char> host(kArgBytes * cnt * B_NKIND);
    for (int kind = 0; kind < B_NKIND; ++kind) {
        char *slot = host.data() + ((char *)G.args_dev[kind] - (char *)G.args_dev[0]);
        const int fam = kFamOf[kind];
        const bool is_lm = (kind == B_KIN_HALF || kind == B_KIN_FULL || kind == B_KERNEL);
        const int N = is_lm ? G.ny : G.nx;
        int var = G.var[fam];
        if (var >= 2 && !uniform) var -= 2;   // same radix plan, one tile per block
        const GKernels *k = gkernels_for(N, var);
        GLaunch L;
        L.pipe = k->pipe && kind != B_ENTRY && kind != B_EXIT;
        L.count = cnt;
        if (is_lm) {
            for (int m = 0; m < cnt; ++m) {
                const LmArgs v = lm_args(b, b->inst[G.members[m]], kind, k->lm_lines, G.var[F_DENSITY]);
                std::memcpy(slot + sizeof(LmArgs) * m, &v, sizeof(v));
                L.tpi = v.s0.ntiles + v.s1.ntiles;   // the same for every member
            }
            L.fn = kind == B_KERNEL ? k->lm_kern : k->lm_kin;
            L.block = dim3(k->lm_threads());
        } else {
            for (int m = 0; m < cnt; ++m) {
                const EmArgs v = em_args(b, b->inst[G.members[m]], kind);
                std::memcpy(slot + sizeof(EmArgs) * m, &v, sizeof(v));
                L.tpi = (v.nlines + k->em_lines - 1) / k->em_lines;
            }
            const bool st = G.store_psi != 0;
            L.fn = kind == B_ENTRY ? k->em_fwd
                 : kind == B_EXIT ? k->em_inv
                 : kind == B_DENSITY ? (st ? k->density_store : k->density)
                                     : (st ? k->phase_real : k->phase);
            L.block = dim3(k->em_threads());
        }
        int grid = L.tpi * cnt;
        if (L.pipe) {
            const int pb = persistent_blocks(L.fn, (int)L.block.x);
            if (pb > 0 && pb < grid) grid = pb;
        }
        L.grid = dim3(grid);
        L.args = G.args_dev[kind];
        if (!(L == G.launch[kind])) b->dirty = true;
        G.launch[kind] = L;
    }
    return upload_sync(b->stream, G.args_dev[0], host.data(), host.size());
}

// Rebuild every group's launch descriptors and upload the argument arrays.
gsn_status build_batch(gsn_batch b)
{
    for (Group &G : b->groups) {
        gsn_status s = build_group(b, G);
        if (s) return s;
    }
    b->q_built = false;
    return GSN_OK;
}

hipError_t glaunch(const GLaunch &L, hipStream_t s)
{
    const void *args_ptr = L.args;
    int tpi = L.tpi, count = L.count;
    void *args[3] = {(void *)&args_ptr, (void *)&tpi, (void *)&count};
    return hipLaunchKernel(L.fn, L.grid, L.block, args, 0, s);
}

// The launch chain of one group for nsteps steps.
gsn_status enqueue_group(const Group &G, int64_t nsteps, hipStream_t s)
{
    HIP_TRY(glaunch(G.launch[B_ENTRY], s));
    HIP_TRY(glaunch(G.launch[B_KIN_HALF], s));
    for (int64_t i = 0; i < nsteps; ++i) {
        HIP_TRY(glaunch(G.launch[B_DENSITY], s));
        HIP_TRY(glaunch(G.launch[B_KERNEL], s));
        HIP_TRY(glaunch(G.launch[B_PHASE], s));
        HIP_TRY(glaunch(G.launch[i + 1 < nsteps ? B_KIN_FULL : B_KIN_HALF], s));
    }
    HIP_TRY(glaunch(G.launch[B_EXIT], s));
    return GSN_OK;
}

gsn_status capture_graph(gsn_batch b, int64_t nsteps)
{
    if (b->exec) {
        // its last launch may still be running
        HIP_TRY(hipStreamSynchronize(b->stream));
        HIP_TRY(hipGraphExecDestroy(b->exec));
        b->exec = nullptr;
    }
    hipEvent_t fork;
    HIP_TRY(hipEventCreateWithFlags(&fork, hipEventDisableTiming));
    std::vector<hipEvent_t> join(b->groups.size());
    for (auto &e : join) HIP_TRY(hipEventCreateWithFlags(&e, hipEventDisableTiming));
    HIP_TRY(hipStreamBeginCapture(b->stream, hipStreamCaptureModeThreadLocal));
    gsn_status st = GSN_OK;
    hipError_t he = hipEventRecord(fork, b->stream);
    for (size_t gi = 0; gi < b->groups.size() && he == hipSuccess && !st; ++gi) {
        he = hipStreamWaitEvent(b->side[gi], fork, 0);
        if (he != hipSuccess) break;
        st = enqueue_group(b->groups[gi], nsteps, b->side[gi]);
        if (st) break;
        he = hipEventRecord(join[gi], b->side[gi]);
        if (he == hipSuccess) he = hipStreamWaitEvent(b->stream, join[gi], 0);
    }
    hipGraph_t graph = nullptr;
    hipError_t ee = hipStreamEndCapture(b->stream, &graph);
    (void)hipEventDestroy(fork);
    for (auto &e : join) (void)hipEventDestroy(e);
    if (st) {
        if (graph) (void)hipGraphDestroy(graph);
        return st;
    }
    if (he != hipSuccess) {
        if (graph) (void)hipGraphDestroy(graph);
        return fail(GSN_EHIP, std::string("graph capture: ") + hipGetErrorString(he));
    }
    if (ee != hipSuccess) return fail(GSN_EHIP, std::string("hipStreamEndCapture: ") + hipGetErrorString(ee));
    hipError_t ie = hipGraphInstantiate(&b->exec, graph, nullptr, nullptr, 0);
    (void)hipGraphDestroy(graph);
    if (ie != hipSuccess) return fail(GSN_EHIP, std::string("hipGraphInstantiate: ") + hipGetErrorString(ie));
    b->exec_steps = nsteps;
    b->dirty = false;
    return GSN_OK;
}

const int kQtoB[Q_NKIND] = {B_ENTRY, B_KIN_HALF, B_DENSITY, B_KERNEL, B_PHASE, B_KIN_FULL, B_EXIT};

template <int N> void ptiles(int nlines_em, int *el, int *ll)
{
    (void)nlines_em;
    *el = PCfg<N>::EL;
    *ll = PCfg<N>::LL;
}

void pcfg_lines(int n, int *el, int *ll)
{
    switch (n) {
    case 128: ptiles<128>(0, el, ll); break;
    case 256: ptiles<256>(0, el, ll); break;
    case 512: ptiles<512>(0, el, ll); break;
    default: ptiles<1024>(0, el, ll); break;
    }
}

// Per-instance tile arguments and per-kind tile prefixes for the persistent kernel.
gsn_status build_persistent(gsn_batch b)
{
    const int count = b->count;
    std::vector<PInst> pin(count);
    std::vector<std::vector<unsigned>> tiles(Q_NKIND, std::vector<unsigned>(count, 0));
    for (int i = 0; i < count; ++i) {
        const Instance &I = b->inst[i];
        if (!persistent_size(I.nx) || !persistent_size(I.ny))
            return fail(GSN_EUNSUPPORTED, "persistent mode supports extents 128..1024");
        int el_x, ll_x, el_y, ll_y;
        pcfg_lines(I.nx, &el_x, &ll_x);
        pcfg_lines(I.ny, &el_y, &ll_y);
        PInst &P = pin[i];
        std::memset(&P, 0, sizeof(P));
        P.nx = I.nx;
        P.ny = I.ny;
        const int dens_tiles = (I.ny / 2 + el_x - 1) / el_x;
        for (int q = 0; q < Q_NKIND; ++q) {
            const int kind = kQtoB[q];
            const bool is_lm = (kind == B_KIN_HALF || kind == B_KIN_FULL || kind == B_KERNEL);
            if (is_lm) {
                P.lm[q] = lm_args(b, I, kind, ll_y, b->var[F_DENSITY]);   // nmass set below
                if (kind == B_KERNEL) P.lm[q].nmass = dens_tiles;
                tiles[q][i] = P.lm[q].s0.ntiles + P.lm[q].s1.ntiles;
            } else {
                P.em[q] = em_args(b, I, kind);
                tiles[q][i] = (P.em[q].nlines + el_x - 1) / el_x;
            }
        }
    }
    // instances to the XCD queues, largest first onto the least loaded queue
    std::vector<int> order(count);
    for (int i = 0; i < count; ++i) order[i] = i;
    std::stable_sort(order.begin(), order.end(), [&](int x, int y) {
        return (long long)b->inst[x].nx * b->inst[x].ny > (long long)b->inst[y].nx * b->inst[y].ny;
    });
    std::vector<std::vector<int>> ql(kNQ);
    long long load[kNQ] = {0};
    for (int i : order) {
        int best = 0;
        for (int x = 1; x < kNQ; ++x)
            if (load[x] < load[best]) best = x;
        ql[best].push_back(i);
        load[best] += (long long)b->inst[i].nx * b->inst[i].ny;
    }
    b->h_prefix.assign(Q_NKIND * (count + kNQ) + count, 0);
    int off = 0;
    for (int x = 0; x < kNQ; ++x) {
        std::sort(ql[x].begin(), ql[x].end());
        const int cx = (int)ql[x].size();
        b->q_count[x] = cx;
        b->q_pre_off[x] = off;
        for (int q = 0; q < Q_NKIND; ++q)
            for (int j = 0; j < cx; ++j)
                b->h_prefix[off + q * (cx + 1) + j + 1] = b->h_prefix[off + q * (cx + 1) + j] + tiles[q][ql[x][j]];
        off += Q_NKIND * (cx + 1);
    }
    for (int x = 0; x < kNQ; ++x) {
        b->q_list_off[x] = off;
        for (int i : ql[x]) b->h_prefix[off++] = (unsigned)i;
    }
    gsn_status s = upload_sync(b->stream, b->q_inst, pin.data(), sizeof(PInst) * count);
    if (s) return s;
    s = upload_sync(b->stream, b->q_prefix, b->h_prefix.data(), 4ull * b->h_prefix.size());
    if (s) return s;
    b->q_built = true;
    return GSN_OK;
}

gsn_status enqueue_persistent(gsn_batch b, int64_t nsteps, hipStream_t st)
{
    PArgs a;
    a.inst = b->q_inst;
    for (int x = 0; x < kNQ; ++x) {
        a.T[x] = QTables{b->q_count[x], (long long)nsteps, b->q_prefix + b->q_pre_off[x]};
        const QTables Th{b->q_count[x], (long long)nsteps, b->h_prefix.data() + b->q_pre_off[x]};
        a.total[x] = b->q_count[x] ? qtotal_items(Th) : 0;
        a.list[x] = (const int *)(b->q_prefix + b->q_list_off[x]);
        b->q_total[x] = a.total[x];
    }
    a.head = b->q_head;
    a.done = b->q_done;
    a.err = b->q_err;
    a.spin_limit = b->spin_limit;
    a.store_psi = b->store_psi;
    a.fail_item = b->fail_item < 0 ? ~0ull : (unsigned long long)b->fail_item;
    int cus = 0;
    HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, b->device));
    hipLaunchKernelGGL(k_queue_reset, dim3((std::max(b->count, kNQ) + 255) / 256), dim3(256), 0, st, b->q_head,
                       b->q_done, b->q_err, b->count);
    hipLaunchKernelGGL(k_batch_persistent, dim3(2 * cus), dim3(kPThreads), 0, st, a);
    HIP_TRY(hipGetLastError());
    return GSN_OK;
}

}  // namespace

// ------------------------------------------------------------------ C ABI
extern "C" gsn_status gsn_batch_workspace_bytes(int count, int ndim, const int32_t *n, size_t *bytes)
{
    gsn_status s = validate_batch(count, ndim, n);
    if (s) return s;
    if (!bytes) return fail(GSN_EINVAL, "bytes is NULL");
    BLayout L;
    compute_blayout(count, n, &L);
    *bytes = L.total;
    return GSN_OK;
}

extern "C" gsn_status gsn_batch_create(gsn_batch *out, int count, int ndim, const int32_t *n,
                                       const double *L, void *d_ws, size_t bytes, void *stream)
{
    if (!out) return fail(GSN_EINVAL, "out is NULL");
    *out = nullptr;
    gsn_status s = validate_batch(count, ndim, n);
    if (s) return s;
    if (!L) return fail(GSN_EINVAL, "L is NULL");
    for (int i = 0; i < 2 * count; ++i)
        if (!(std::isfinite(L[i]) && L[i] > 0.0)) return fail(GSN_EINVAL, "box lengths must be finite and > 0");
    if (!d_ws) return fail(GSN_EINVAL, "workspace is NULL");
    if (((uintptr_t)d_ws & 255) != 0) return fail(GSN_EWORKSPACE, "workspace must be 256-byte aligned");
    BLayout lay;
    compute_blayout(count, n, &lay);
    if (bytes < lay.total)
        return fail(GSN_EWORKSPACE, "workspace too small: need " + std::to_string(lay.total) + " bytes");
    gsn_batch b = new (std::nothrow) gsn_batch_();
    if (!b) return fail(GSN_EINVAL, "out of host memory");
    b->count = count;
    b->user = (hipStream_t)stream;
    if (hipStreamCreateWithFlags(&b->stream, hipStreamNonBlocking) != hipSuccess ||
        hipEventCreateWithFlags(&b->ev_in, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&b->ev_out, hipEventDisableTiming) != hipSuccess) {
        delete b;
        return fail(GSN_EHIP, "stream/event creation failed");
    }
    b->ws = (char *)d_ws;
    b->ws_bytes = bytes;
    b->exec = nullptr;
    b->exec_steps = -1;
    b->dirty = true;
    b->mode = 0;
    b->store_psi = 1;
    b->pq = b->ws + lay.queue_off;
    {
        char *q = (char *)b->pq;
        b->q_head = (unsigned long long *)q;
        b->q_err = (unsigned *)(q + 64);
        q += align256(256);
        b->q_done = (unsigned long long *)q;
        q += align256(8ull * count);
        b->q_prefix = (unsigned *)q;
        q += align256(4ull * (Q_NKIND * (count + kNQ) + count));
        b->q_inst = (PInst *)q;
        b->q_built = false;
        for (int x = 0; x < kNQ; ++x) {
            b->q_count[x] = b->q_pre_off[x] = b->q_list_off[x] = 0;
            b->q_total[x] = 0;
        }
        b->spin_limit = 1u << 22;
        b->fail_item = -1;
    }
    // default schedule: the fastest measured on gfx950 for the 64-instance
    // sweep of 256^2 / 512^2 / 1024^2 grids (persistent passes, real-space
    // psi stored by the density pass)
    b->var[F_KIN] = 2;
    b->var[F_DENSITY] = 3;
    b->var[F_KERNEL] = 2;
    b->var[F_PHASE] = 3;
    b->var[F_XFFT] = 0;
    if (hipGetDevice(&b->device) != hipSuccess) {
        delete b;
        return fail(GSN_EHIP, "hipGetDevice failed");
    }
    b->scratch = (float2 *)(b->ws + lay.scratch_off);
    b->scratch_bytes = lay.scratch_bytes;
    b->st = b->ws + lay.st_off;
    b->k2_unit = (double *)(b->ws + lay.unit_off);
    b->kin_unit = (double2 *)(b->ws + lay.unit_off + 256);
    b->sct = (double2 *)(b->ws + lay.unit_off + 512);
    b->inst.resize(count);
    std::map<std::pair<int, int>, int> gidx;
    for (int i = 0; i < count; ++i) {
        Instance &I = b->inst[i];
        std::memset(&I, 0, sizeof(I));
        I.ny = n[2 * i];
        I.nx = n[2 * i + 1];
        I.Ly = L[2 * i];
        I.Lx = L[2 * i + 1];
        I.P = (long long)I.ny * I.nx;
        I.a = 0.5;
        char *p = b->ws + lay.inst_off[i];
        int db = 0;
        for (int v = 0; v < kNumVariants; ++v) {
            const NKernels *k = kernels_for(I.nx, v);
            db = std::max(db, (int)((I.ny / 2 + k->em_lines - 1) / k->em_lines));
        }
        const int M = std::max(I.nx, I.ny);
        I.psi = (float2 *)p; p += align256(8ull * I.P);
        I.half = (float2 *)p; p += align256(4ull * I.P);
        I.nyq = (float2 *)p; p += align256(8ull * I.ny);
        I.mass_parts = (double *)p; p += align256(8ull * db);
        I.st = (DevState *)(b->st + kStateStride * i);
        I.tw_x = (double2 *)p; p += align256(16ull * M);
        I.tw_y = (double2 *)p; p += align256(16ull * M);
        I.kinF_x = (double2 *)p; p += align256(16ull * M);
        I.kinF_y = (double2 *)p; p += align256(16ull * M);
        I.kinH_x = (double2 *)p; p += align256(16ull * M);
        I.kinH_y = (double2 *)p; p += align256(16ull * M);
        I.k2_x = (double *)p; p += align256(8ull * M);
        I.k2_y = (double *)p; p += align256(8ull * M);
        auto key = std::make_pair(I.ny, I.nx);
        if (!gidx.count(key)) {
            gidx[key] = (int)b->groups.size();
            Group G{};
            G.ny = I.ny;
            G.nx = I.nx;
            for (int f = 0; f < F_NFAM; ++f) G.var[f] = b->var[f];
            G.store_psi = b->store_psi;
            b->groups.push_back(G);
        }
        b->groups[gidx[key]].members.push_back(i);
    }
    // argument arrays: per group, per kind, one slot per member
    {
        char *p = b->ws + lay.args_off;
        for (Group &G : b->groups)
            for (int kind = 0; kind < B_NKIND; ++kind) {
                G.args_dev[kind] = p;
                p += kArgBytes * G.members.size();
            }
    }
    const double zero = 0.0;
    const double2 one = make_double2(1.0, 0.0);
    std::vector<double2> sct(kSinCosTable);
    fill_sincos_table(sct.data());
    if ((s = upload_sync(b->stream, b->k2_unit, &zero, 8)) || (s = upload_sync(b->stream, b->kin_unit, &one, 16)) ||
        (s = upload_sync(b->stream, b->sct, sct.data(), 16ull * kSinCosTable))) {
        delete b;
        return s;
    }
    b->side.resize(b->groups.size());
    for (auto &st : b->side)
        if (hipStreamCreateWithFlags(&st, hipStreamNonBlocking) != hipSuccess) {
            for (auto &x : b->side)
                if (x) (void)hipStreamDestroy(x);
            delete b;
            return fail(GSN_EHIP, "hipStreamCreate failed");
        }
    for (Instance &I : b->inst) {
        if ((s = upload_instance_tables(b, I))) {
            for (auto &x : b->side) (void)hipStreamDestroy(x);
            delete b;
            return s;
        }
        hipLaunchKernelGGL(k_reset_state, dim3(1), dim3(64), 0, b->stream, I.st);
    }
    if ((s = build_batch(b))) {
        for (auto &x : b->side) (void)hipStreamDestroy(x);
        delete b;
        return s;
    }
    *out = b;
    return GSN_OK;
}

extern "C" gsn_status gsn_batch_destroy(gsn_batch b)
{
    if (!b) return fail(GSN_EINVAL, "batch is NULL");
    (void)hipStreamSynchronize(b->stream);
    if (b->exec) (void)hipGraphExecDestroy(b->exec);
    for (auto &x : b->side) (void)hipStreamDestroy(x);
    (void)hipEventDestroy(b->ev_in);
    (void)hipEventDestroy(b->ev_out);
    (void)hipStreamDestroy(b->stream);
    delete b;
    return GSN_OK;
}

extern "C" gsn_status gsn_batch_set(gsn_batch b, int i, const gsn_kernel *k, double a_kin, double g_local,
                                    double dz, const void *psi, int on_device, int dtype)
{
    if (!b || !k || !psi) return fail(GSN_EINVAL, "NULL argument");
    if (i < 0 || i >= b->count) return fail(GSN_EINVAL, "instance index out of range");
    if (dtype != GSN_C64 && dtype != GSN_C128) return fail(GSN_EINVAL, "dtype must be GSN_C64 or GSN_C128");
    if (!std::isfinite(k->c_newton) || !std::isfinite(k->c_yukawa) || !std::isfinite(k->m_yukawa) ||
        !std::isfinite(k->c_contact))
        return fail(GSN_EINVAL, "kernel coefficients must be finite");
    if (k->c_yukawa != 0.0 && !(k->m_yukawa > 0.0)) return fail(GSN_EINVAL, "m_yukawa must be > 0 when c_yukawa != 0");
    if (!std::isfinite(a_kin) || !std::isfinite(g_local) || !std::isfinite(dz) || dz == 0.0)
        return fail(GSN_EINVAL, "coefficients must be finite and dz != 0");
    HIP_TRY(hipSetDevice(b->device));
    HIP_TRY(hipStreamSynchronize(b->stream));
    Instance &I = b->inst[i];
    I.kern = *k;
    I.a = a_kin;
    I.g = g_local;
    I.dz = dz;
    gsn_status s = upload_instance_tables(b, I);
    if (s) return s;
    if (dtype == GSN_C64) {
        HIP_TRY(hipMemcpyAsync(I.psi, psi, 8ull * I.P, on_device ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice,
                               b->stream));
    } else if (on_device) {
        hipLaunchKernelGGL(k_from_c128, dim3(1024), dim3(256), 0, b->stream, (const double2 *)psi, I.psi, I.P);
        HIP_TRY(hipGetLastError());
    } else {
        std::vector<float2> tmp((size_t)I.P);
        const double *src = (const double *)psi;
        for (long long q = 0; q < I.P; ++q) tmp[q] = make_float2((float)src[2 * q], (float)src[2 * q + 1]);
        HIP_TRY(hipMemcpyAsync(I.psi, tmp.data(), 8ull * I.P, hipMemcpyHostToDevice, b->stream));
        HIP_TRY(hipStreamSynchronize(b->stream));
    }
    hipLaunchKernelGGL(k_reset_state, dim3(1), dim3(64), 0, b->stream, I.st);
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipStreamSynchronize(b->stream));
    I.set = true;
    b->q_built = false;
    for (Group &G : b->groups)   // only its own group reads the instance
        if (G.ny == I.ny && G.nx == I.nx) return build_group(b, G);
    return fail(GSN_EINVAL, "instance not in any group");
}

extern "C" gsn_status gsn_batch_step(gsn_batch b, int64_t nsteps)
{
    if (!b) return fail(GSN_EINVAL, "batch is NULL");
    if (nsteps < 0) return fail(GSN_EINVAL, "nsteps must be >= 0");
    for (const Instance &I : b->inst)
        if (!I.set) return fail(GSN_ESTATE, "every instance must be set before stepping");
    if (nsteps == 0) return GSN_OK;
    HIP_TRY(hipSetDevice(b->device));
    // order after the caller's earlier work, run on the internal stream, and
    // make the caller's later work wait for the run
    HIP_TRY(hipEventRecord(b->ev_in, b->user));
    HIP_TRY(hipStreamWaitEvent(b->stream, b->ev_in, 0));
    if (b->mode == 0) {
        if (b->dirty || !b->exec || b->exec_steps != nsteps) {
            gsn_status s = capture_graph(b, nsteps);
            if (s) return s;
        }
        HIP_TRY(hipGraphLaunch(b->exec, b->stream));
    } else if (b->mode == 1) {
        if (!b->q_built) {
            gsn_status s = build_persistent(b);
            if (s) return s;
        }
        gsn_status s = enqueue_persistent(b, nsteps, b->stream);
        if (s) return s;
    } else {
        // mode 2: the same grouped launches issued directly (no graph)
        for (size_t gi = 0; gi < b->groups.size(); ++gi) {
            gsn_status s = enqueue_group(b->groups[gi], nsteps, b->stream);
            if (s) return s;
        }
    }
    HIP_TRY(hipEventRecord(b->ev_out, b->stream));
    HIP_TRY(hipStreamWaitEvent(b->user, b->ev_out, 0));
    return GSN_OK;
}

extern "C" gsn_status gsn_batch_sync(gsn_batch b)
{
    if (!b) return fail(GSN_EINVAL, "batch is NULL");
    HIP_TRY(hipSetDevice(b->device));
    HIP_TRY(hipStreamSynchronize(b->stream));
    HIP_TRY(hipStreamSynchronize(b->user));
    if (b->mode == 1) {
        unsigned err = 0;
        HIP_TRY(hipMemcpy(&err, b->q_err, 4, hipMemcpyDeviceToHost));
        if (err) return fail(GSN_EHIP, "persistent batch queue: a wait exceeded its spin limit");
        unsigned long long head[kNQ];
        HIP_TRY(hipMemcpy(head, b->q_head, sizeof(head), hipMemcpyDeviceToHost));
        for (int x = 0; x < kNQ; ++x)
            if (b->q_count[x] && head[x] < b->q_total[x])
                return fail(GSN_EHIP, "persistent batch queue: an XCD's queue was not drained (no block ran there)");
    }
    std::vector<char> all(kStateStride * b->count);
    HIP_TRY(hipMemcpy(all.data(), b->st, all.size(), hipMemcpyDeviceToHost));
    for (int i = 0; i < b->count; ++i) {
        DevState st;
        std::memcpy(&st, all.data() + kStateStride * i, sizeof(st));
        if (st.nonfinite) return fail(GSN_ENONFINITE, "an instance's fused FP64 mass became non-finite");
    }
    return GSN_OK;
}

extern "C" gsn_status gsn_batch_get(gsn_batch b, int i, void *dst, int on_device, int dtype)
{
    if (!b || !dst) return fail(GSN_EINVAL, "NULL argument");
    if (i < 0 || i >= b->count) return fail(GSN_EINVAL, "instance index out of range");
    if (dtype != GSN_C64 && dtype != GSN_C128) return fail(GSN_EINVAL, "dtype must be GSN_C64 or GSN_C128");
    HIP_TRY(hipSetDevice(b->device));
    const Instance &I = b->inst[i];
    const size_t esz = dtype == GSN_C128 ? 16 : 8;
    void *out = on_device ? dst : (void *)b->scratch;
    if (dtype == GSN_C128)
        hipLaunchKernelGGL(k_readout<true>, dim3(1024), dim3(256), 0, b->stream, I.psi, out, I.P, I.st);
    else
        hipLaunchKernelGGL(k_readout<false>, dim3(1024), dim3(256), 0, b->stream, I.psi, out, I.P, I.st);
    HIP_TRY(hipGetLastError());
    if (!on_device) HIP_TRY(hipMemcpyAsync(dst, b->scratch, esz * I.P, hipMemcpyDeviceToHost, b->stream));
    HIP_TRY(hipStreamSynchronize(b->stream));
    return gsn_batch_sync(b);
}

extern "C" gsn_status gsn_batch_mass(gsn_batch b, double *masses)
{
    if (!b || !masses) return fail(GSN_EINVAL, "NULL argument");
    HIP_TRY(hipSetDevice(b->device));
    const int per = (int)std::min<size_t>(b->scratch_bytes / (8 * kMassParts), (size_t)b->count);
    double *parts = (double *)b->scratch;
    std::vector<double> h((size_t)per * kMassParts);
    for (int i0 = 0; i0 < b->count; i0 += per) {
        const int n = std::min(per, b->count - i0);
        for (int j = 0; j < n; ++j) {
            const Instance &I = b->inst[i0 + j];
            hipLaunchKernelGGL(k_mass<256>, dim3(kMassParts), dim3(256), 0, b->stream, I.psi, I.P,
                               parts + (size_t)j * kMassParts);
            HIP_TRY(hipGetLastError());
        }
        HIP_TRY(hipMemcpyAsync(h.data(), parts, 8ull * kMassParts * n, hipMemcpyDeviceToHost, b->stream));
        HIP_TRY(hipStreamSynchronize(b->stream));
        for (int j = 0; j < n; ++j) {
            const Instance &I = b->inst[i0 + j];
            double sum = 0.0;
            for (int q = 0; q < kMassParts; ++q) sum += h[(size_t)j * kMassParts + q];
            masses[i0 + j] = sum * (I.Lx / I.nx) * (I.Ly / I.ny);
        }
    }
    return gsn_batch_sync(b);
}

extern "C" gsn_status gsn_batch_set_mode(gsn_batch b, int mode)
{
    if (!b) return fail(GSN_EINVAL, "batch is NULL");
    if (mode != 0 && mode != 1 && mode != 2)
        return fail(GSN_EINVAL, "mode must be 0 (graph), 1 (persistent) or 2 (direct launches)");
    if (mode == 1) {
        HIP_TRY(hipSetDevice(b->device));
        gsn_status s = build_persistent(b);
        if (s) return s;
    }
    b->mode = mode;
    return GSN_OK;
}

extern "C" gsn_status gsn_batch_set_schedule(gsn_batch b, const int *variants, int nfam, int nonlinear_mode)
{
    if (!b || !variants || nfam < F_NFAM) return fail(GSN_EINVAL, "bad schedule arguments");
    for (int i = 0; i < F_NFAM; ++i)
        if (variants[i] < 0 || variants[i] >= kNumBatchVariants) return fail(GSN_EINVAL, "unknown schedule variant");
    if (nonlinear_mode != 0 && nonlinear_mode != 1) return fail(GSN_EINVAL, "nonlinear mode must be 0 or 1");
    HIP_TRY(hipSetDevice(b->device));
    HIP_TRY(hipStreamSynchronize(b->stream));
    for (int i = 0; i < F_NFAM; ++i) b->var[i] = variants[i];
    b->store_psi = nonlinear_mode;
    for (Group &G : b->groups) {
        for (int i = 0; i < F_NFAM; ++i) G.var[i] = variants[i];
        G.store_psi = nonlinear_mode;
    }
    return build_batch(b);
}

// ---------------------------------------------------------------- batch autotuner
namespace {

// Average time of one step of a group's chain (density, kernel, phase,
// kinetic), or of one entry + exit transform pair (xfft), over iters
// repetitions after one untimed one, on the batch's stream.
gsn_status time_group(gsn_batch b, Group &G, int iters, bool xfft, double *ms)
{
    gsn_status s = build_group(b, G);
    if (s) return s;
    auto chain = [&]() -> hipError_t {
        hipError_t e = hipSuccess;
        if (xfft) {
            if ((e = glaunch(G.launch[B_ENTRY], b->stream)) != hipSuccess) return e;
            return glaunch(G.launch[B_EXIT], b->stream);
        }
        const int kinds[4] = {B_DENSITY, B_KERNEL, B_PHASE, B_KIN_FULL};
        for (int k : kinds)
            if ((e = glaunch(G.launch[k], b->stream)) != hipSuccess) return e;
        return e;
    };
    hipEvent_t e0, e1;
    HIP_TRY(hipEventCreate(&e0));
    HIP_TRY(hipEventCreate(&e1));
    hipError_t he = chain();
    if (he == hipSuccess) he = hipEventRecord(e0, b->stream);
    for (int i = 0; i < iters && he == hipSuccess; ++i) he = chain();
    if (he == hipSuccess) he = hipEventRecord(e1, b->stream);
    if (he == hipSuccess) he = hipEventSynchronize(e1);
    float t = 0.f;
    if (he == hipSuccess) he = hipEventElapsedTime(&t, e0, e1);
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (he != hipSuccess) return fail(GSN_EHIP, std::string("batch autotune timing: ") + hipGetErrorString(he));
    *ms = (double)t / iters;
    return GSN_OK;
}

std::string batch_cache_key(gsn_batch b, const Group &G, const char *what)
{
    hipDeviceProp_t prop;
    std::string arch = "unknown";
    if (hipGetDeviceProperties(&prop, b->device) == hipSuccess) arch = prop.gcnArchName;
    const size_t colon = arch.find(':');
    if (colon != std::string::npos) arch = arch.substr(0, colon);
    return arch + " batch 2d " + std::to_string(G.ny) + "x" + std::to_string(G.nx) + " " + what;
}

const char *kFamNames[F_NFAM] = {"kinetic", "x_density", "kernel", "x_phase", "x_fft"};

// Choose the fastest variant of family fam for group G (others fixed).
gsn_status tune_family(gsn_batch b, Group &G, int fam, int iters, double *best_ms)
{
    int best = G.var[fam];
    double bms = 1e300;
    for (int v = 0; v < kNumBatchVariants; ++v) {
        G.var[fam] = v;
        double ms = 0.0;
        gsn_status s = time_group(b, G, iters, fam == F_XFFT, &ms);
        if (s) return s;
        if (ms < bms) { bms = ms; best = v; }
    }
    G.var[fam] = best;
    *best_ms = bms;
    return GSN_OK;
}

}  // namespace

extern "C" gsn_status gsn_batch_autotune(gsn_batch b, int iters)
{
    if (!b) return fail(GSN_EINVAL, "batch is NULL");
    if (iters < 1 || iters > 10000) return fail(GSN_EINVAL, "iters must be in [1, 10000]");
    for (const Instance &I : b->inst)
        if (!I.set) return fail(GSN_ESTATE, "every instance must be set before autotuning");
    HIP_TRY(hipSetDevice(b->device));
    HIP_TRY(hipStreamSynchronize(b->user));
    HIP_TRY(hipStreamSynchronize(b->stream));
    // the timed passes run in place on the instances' buffers (realistic
    // data, bounded: whole split steps, and forward / inverse transform
    // pairs); the states are saved to host memory and put back at the end
    std::vector<std::vector<float2>> keep(b->count);
    std::vector<DevState> keep_st(b->count);
    for (int i = 0; i < b->count; ++i) {
        const Instance &I = b->inst[i];
        keep[i].resize((size_t)I.P);
        HIP_TRY(hipMemcpyAsync(keep[i].data(), I.psi, 8ull * I.P, hipMemcpyDeviceToHost, b->stream));
        HIP_TRY(hipMemcpyAsync(&keep_st[i], I.st, sizeof(DevState), hipMemcpyDeviceToHost, b->stream));
    }
    HIP_TRY(hipStreamSynchronize(b->stream));
    const char *cpath = std::getenv("GSN_AUTOTUNE_CACHE");
    std::map<std::string, int> cache;
    if (cpath && *cpath) {
        std::ifstream f(cpath);
        std::string line;
        while (std::getline(f, line)) {
            const size_t sp = line.rfind(' ');
            if (sp == std::string::npos) continue;
            cache[line.substr(0, sp)] = std::atoi(line.c_str() + sp + 1);
        }
    }
    std::vector<std::string> fresh;
    gsn_status s = GSN_OK;
    for (Group &G : b->groups) {
        bool cached = true;
        int cv[F_NFAM], cm = 0;
        for (int f = 0; f < F_NFAM && cached; ++f) {
            auto it = cache.find(batch_cache_key(b, G, kFamNames[f]));
            cached = it != cache.end() && it->second >= 0 && it->second < kNumBatchVariants;
            if (cached) cv[f] = it->second;
        }
        auto mit = cache.find(batch_cache_key(b, G, "nonlinear_mode"));
        cached = cached && mit != cache.end() && (mit->second == 0 || mit->second == 1);
        if (cached) {
            cm = mit->second;
            for (int f = 0; f < F_NFAM; ++f) G.var[f] = cv[f];
            G.store_psi = cm;
            continue;
        }
        double ms = 0.0;
        // the column passes do not depend on the nonlinear mode
        if ((s = tune_family(b, G, F_KIN, iters, &ms)) || (s = tune_family(b, G, F_KERNEL, iters, &ms))) break;
        // the density and phase passes change together with the mode
        int bv[2][2];
        double bm[2];
        for (int m = 0; m < 2 && !s; ++m) {
            G.store_psi = m;
            if ((s = tune_family(b, G, F_DENSITY, iters, &ms)) || (s = tune_family(b, G, F_PHASE, iters, &ms)))
                break;
            bv[m][0] = G.var[F_DENSITY];
            bv[m][1] = G.var[F_PHASE];
            bm[m] = ms;
        }
        if (s) break;
        const int m = bm[1] < bm[0] ? 1 : 0;
        G.store_psi = m;
        G.var[F_DENSITY] = bv[m][0];
        G.var[F_PHASE] = bv[m][1];
        if ((s = tune_family(b, G, F_XFFT, iters, &ms))) break;
        for (int f = 0; f < F_NFAM; ++f)
            fresh.push_back(batch_cache_key(b, G, kFamNames[f]) + " " + std::to_string(G.var[f]));
        fresh.push_back(batch_cache_key(b, G, "nonlinear_mode") + " " + std::to_string(G.store_psi));
    }
    // put the states back (also after a failed timing)
    for (int i = 0; i < b->count; ++i) {
        const Instance &I = b->inst[i];
        HIP_TRY(hipMemcpyAsync(I.psi, keep[i].data(), 8ull * I.P, hipMemcpyHostToDevice, b->stream));
        HIP_TRY(hipMemcpyAsync(I.st, &keep_st[i], sizeof(DevState), hipMemcpyHostToDevice, b->stream));
    }
    HIP_TRY(hipStreamSynchronize(b->stream));
    if (s) return s;
    if ((s = build_batch(b))) return s;
    if (cpath && *cpath && !fresh.empty()) {
        std::ofstream f(cpath, std::ios::app);
        for (const std::string &l : fresh) f << l << "\n";
    }
    return GSN_OK;
}

extern "C" gsn_status gsn_batch_get_schedule(gsn_batch b, int i, int *variants, int nfam, int *nonlinear_mode)
{
    if (!b || !variants || !nonlinear_mode || nfam < F_NFAM) return fail(GSN_EINVAL, "bad schedule arguments");
    if (i < 0 || i >= b->count) return fail(GSN_EINVAL, "instance index out of range");
    for (const Group &G : b->groups)
        for (int m : G.members)
            if (m == i) {
                for (int f = 0; f < F_NFAM; ++f) variants[f] = G.var[f];
                *nonlinear_mode = G.store_psi;
                return GSN_OK;
            }
    return fail(GSN_EINVAL, "instance not in any group");
}

extern "C" gsn_status gsn_batch_phase(gsn_batch b, int i, double *theta, int64_t *steps)
{
    if (!b) return fail(GSN_EINVAL, "batch is NULL");
    if (i < 0 || i >= b->count) return fail(GSN_EINVAL, "instance index out of range");
    HIP_TRY(hipSetDevice(b->device));
    HIP_TRY(hipStreamSynchronize(b->stream));
    DevState st;
    HIP_TRY(hipMemcpy(&st, b->inst[i].st, sizeof(st), hipMemcpyDeviceToHost));
    if (theta) *theta = st.theta;
    if (steps) *steps = st.steps;
    return GSN_OK;
}

extern "C" gsn_status gsn_batch_set_queue_limits(gsn_batch b, unsigned spin_limit, long long fail_item)
{
    if (!b) return fail(GSN_EINVAL, "batch is NULL");
    if (spin_limit < 1) return fail(GSN_EINVAL, "spin_limit must be >= 1");
    b->spin_limit = spin_limit;
    b->fail_item = fail_item;
    return GSN_OK;
}
