// gsn_small.hpp -- the passes of a split step for grids too small to fill the
// chip (schedule variant "s4").
//
// On such grids a pass is a chain of latencies, not bytes or instructions: at
// 128^2 no SIMD holds more than one wave and a pass takes about 5 us, of which
// 2.4 us is the launch itself.  These tiles shorten the chain:
//   * 4 points per thread up to 256-point lines, so twice the waves of the
//     8-point forms share the arithmetic (from 512 points on one more exchange
//     would cost more than that saves);
//   * complex128 LDS slots: no conversions around an exchange, and nothing is
//     rounded between the stages of a transform;
//   * both rows of a pair are transformed together, sharing twiddles and
//     exchanges, so each row's dependent instructions fill the other's gaps;
//   * every global load of a tile is issued before its first transform;
//   * the sum of the mass partials has a block of its own.
// A step of 128^2 takes 18.8 us with them (22.2 with s8, the best before), one
// of 256^2 19.7 (24.3), of 512^2 28.3 (30.3), of 64^3 31.1 (36.0).
#pragma once
#include "gsn_kernels.hpp"

namespace gsn {

// points per thread of an s4 line, and the lines of a block
template <int N> struct SmCfg {
    static constexpr int E0 = N >= 512 ? 8 : 4;
    static constexpr int E = N < E0 ? N : E0;
    static constexpr int TPL = N / E;
    static constexpr int WLINES = TPL >= 64 ? 1 : 64 / TPL;   // rows or row pairs of an x block
    static constexpr int NT = 256;                            // threads of a strided block
    static constexpr int LINES = NT / TPL;                    // its lines
};

template <int E, int TPL, class ST>
__device__ __forceinline__ void sm_load_line(const ST *q, const ST *safe, long long es, bool act, int t, ST (&raw)[E])
{
    const ST *src = act ? q : safe;
#pragma unroll
    for (int e = 0; e < E; ++e) raw[e] = src[(long long)(t + TPL * e) * es];
}
template <int E, class ST> __device__ __forceinline__ void sm_widen(const ST (&raw)[E], bool act, dc (&v)[E])
{
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = act ? ld_c(raw[e]) : mk(0.0, 0.0);
}

// NB lines transformed together (line b exchanges through lds + b stride): the
// stages of fft_stages, with one twiddle read and one exchange for all of them.
// Values stored as complex64 (ST) take the shorter butterflies.
template <int NB, int N, int E, int S, int ST, bool FULL, class Lay>
__device__ __forceinline__ void sm_stages(dc (&v)[NB][E], int t, const Lay &lay, double2 *lds, int stride,
                                          const double2 *__restrict__ tw)
{
    using P = Plan<N, E>;
    if constexpr (ST < P::nstages()) {
        constexpr int R = P::radix(ST), NS = P::ns(ST), B = E / R, TPL = P::TPL;
        constexpr bool LAST = (ST + 1 == P::nstages());
#pragma unroll
        for (int m = 0; m < B; ++m) {
            const int j = t + TPL * m;
            dc w[R];   // shared by the NB lines
            const Twiddles<N / (NS * R), S> tws{tw, j & (NS - 1)};
            if constexpr (NS > 1) {
#pragma unroll
                for (int r = 1; r < R; ++r) w[r] = tws(r);
            }
            const int base = (j / NS) * NS * R + (j & (NS - 1));
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                dc a[R];
#pragma unroll
                for (int r = 0; r < R; ++r) a[r] = v[b][m + r * B];
                dft<R, S, (NS > 1), FULL>(a, [&](int r) { return w[r]; });
                if constexpr (LAST) {
#pragma unroll
                    for (int r = 0; r < R; ++r) v[b][m + r * B] = a[r];
                } else {
#pragma unroll
                    for (int r = 0; r < R; ++r) lds_put(lds + b * stride, lay(base + r * NS), a[r]);
                }
            }
        }
        if constexpr (!LAST) {
            exchange_sync<Lay::WAVE_LOCAL>();
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int e = 0; e < E; ++e) v[b][e] = lds_get(lds + b * stride, lay(t + TPL * e));
            exchange_sync<Lay::WAVE_LOCAL>();
            sm_stages<NB, N, E, S, ST + 1, FULL>(v, t, lay, lds, stride, tw);
        }
    }
}
template <int NB, int N, int E, int S, class ST, class Lay>
__device__ __forceinline__ void sm_fft(dc (&v)[NB][E], int t, const Lay &lay, double2 *lds, int stride,
                                       const double2 *__restrict__ tw)
{
    sm_stages<NB, N, E, S, 0, kFullFp64<ST>>(v, t, lay, lds, stride, tw);
}

// slots of an x block of LINES pairs (two rows per pair)
template <int N, int LINES> constexpr int sm_em_slots() { return 2 * LINES * EmLayout<N, SmCfg<N>::E>::PITCH; }
template <int N, int LINES> constexpr int sm_lm_slots() { return LINES * N; }

// Row FFT (entry / exit).
template <int N, int LINES, int S, class ST>
__device__ __forceinline__ void sm_em_fft(const EmArgs &a, int tile, const double2 *tw, double2 *lds)
{
    constexpr int E = SmCfg<N>::E, TPL = N / E;
    const int tid = threadIdx.x, t = tid % TPL, l = tid / TPL;
    const int row = tile * LINES + l;
    const bool act = row < a.nlines;
    const EmLayout<N, E> lay{l * EmLayout<N, E>::PITCH};
    ST *p = (ST *)a.psi + (long long)row * N;
    ST raw[E];
    dc v[1][E];
    sm_load_line<E, TPL>(p, (const ST *)a.psi, 1, act, t, raw);
    sm_widen<E>(raw, act, v[0]);
    sm_fft<1, N, E, S, ST>(v, t, lay, lds, 0, tw);
    if (act) {
#pragma unroll
        for (int e = 0; e < E; ++e) p[t + TPL * e] = st_c<ST>(scl(v[0][e], a.scale));
    }
}

// Density pass (as density_tile), one mass partial per wave.
template <int N, int LINES, bool STORE_PSI, class ST>
__device__ __forceinline__ void sm_density(const EmArgs &a, int tile, const double2 *tw, double2 *lds)
{
    constexpr int E = SmCfg<N>::E, TPL = N / E, NT = LINES * TPL, WAVES = (NT + 63) / 64;
    constexpr int STRIDE = LINES * EmLayout<N, E>::PITCH;
    const int tid = threadIdx.x, t = tid % TPL, l = tid / TPL;
    const int pair = tile * LINES + l;
    const bool act = pair < a.nlines;
    const EmLayout<N, E> lay{l * EmLayout<N, E>::PITCH};
    const long long r0 = 2LL * pair, r1 = r0 + 1;
    const double inv_n = 1.0 / N;
    ST *p0 = (ST *)a.psi + r0 * N, *p1 = p0 + N;
    ST q0[E], q1[E];
    dc v[2][E];
    sm_load_line<E, TPL>(p0, (const ST *)a.psi, 1, act, t, q0);
    sm_load_line<E, TPL>(p1, (const ST *)a.psi, 1, act, t, q1);
    sm_widen<E>(q0, act, v[0]);
    sm_widen<E>(q1, act, v[1]);
    sm_fft<2, N, E, 1, ST>(v, t, lay, lds, STRIDE, tw);
    if constexpr (STORE_PSI) {
        if (act) {
            ST *s0 = (ST *)(a.psi_st ? a.psi_st : a.psi) + r0 * N, *s1 = s0 + N;
#pragma unroll
            for (int e = 0; e < E; ++e) {
                s0[t + TPL * e] = st_c<ST>(scl(v[0][e], inv_n));
                s1[t + TPL * e] = st_c<ST>(scl(v[1][e], inv_n));
            }
        }
    }
    double msum = 0.0;
    dc z[1][E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const double rho0 = norm2(v[0][e]) * (inv_n * inv_n), rho1 = norm2(v[1][e]) * (inv_n * inv_n);
        msum += rho0 + rho1;
        z[0][e] = mk(rho0, rho1);
    }
    sm_fft<1, N, E, -1, ST>(z, t, lay, lds, 0, tw);
    store_real_pair<N, E>(z[0], act, t, lay, lds, (ST *)a.half, (ST *)a.nyq, r0, r1);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) msum += __shfl_xor(msum, o, 64);
    if ((tid & 63) == 0) a.partials[tile * WAVES + (tid >> 6)] = msum;
}

// The spectrum of two real rows packed as one complex line (as load_real_pair),
// loaded raw and put together after other loads have been issued.
template <int N, int E, class ST>
__device__ __forceinline__ void sm_load_pair(const ST *half, const ST *nyq, long long r0, int t, ST (&a0)[E],
                                             ST (&a1)[E], ST &n0, ST &n1)
{
    const ST *h0 = half + r0 * (N / 2), *h1 = h0 + N / 2;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int k = t + (N / E) * e;
        const int idx = e < E / 2 ? k : (N - k) & (N / 2 - 1);   // the Nyquist lane reads bin 0
        a0[e] = h0[idx];
        a1[e] = h1[idx];
    }
    n0 = nyq[r0];
    n1 = nyq[r0 + 1];
}
template <int N, int E, class ST>
__device__ __forceinline__ void sm_join_pair(const ST (&a0)[E], const ST (&a1)[E], const ST &n0, const ST &n1, int t,
                                             dc (&z)[E])
{
#pragma unroll
    for (int e = 0; e < E; ++e) {
        dc x0 = ld_c(a0[e]), x1 = ld_c(a1[e]);
        if (e < E / 2) {
            if (t + (N / E) * e == 0) { x0.y = 0.0; x1.y = 0.0; }
        } else if (e == E / 2 && t == 0) {
            x0 = mk(ld_c(n0).x, 0.0);
            x1 = mk(ld_c(n1).x, 0.0);
        } else {
            x0 = conj(x0);
            x1 = conj(x1);
        }
        z[e] = mk(x0.x - x1.y, x0.y + x1.x);
    }
}

// Phase pass (as phase_tile without ENERGY, phi kept in FP64).  LOCAL: with the
// local terms and the static potential, as phase_local_tile: the spectrum of
// lap(s) and the potential's rows are loaded with everything else, ahead of the
// first transform (a step with pressure and Bohm term against the one-tile pass:
// 64x128 25.9 -> 24.6 us, 64x2048 55.6 -> 52.6, 64x128x64 67.6 -> 63.6).
template <int N, int LINES, bool REAL_IN, bool LOCAL, class ST>
__device__ __forceinline__ void sm_phase(const EmArgs &a, int tile, const double2 *tw,
                                         const double2 *sct, double2 *lds)
{
    constexpr int E = SmCfg<N>::E, TPL = N / E, STRIDE = LINES * EmLayout<N, E>::PITCH;
    const int tid = threadIdx.x, t = tid % TPL, l = tid / TPL;
    const int pair = tile * LINES + l;
    const bool act = pair < a.nlines;
    const EmLayout<N, E> lay{l * EmLayout<N, E>::PITCH};
    const long long r0 = act ? 2LL * pair : 0, r1 = r0 + 1;
    const double inv_n = 1.0 / N;
    ST *p0 = (ST *)a.psi + r0 * N, *p1 = p0 + N;
    ST a0[E], a1[E], n0, n1, b0[E], b1[E], m0, m1, q0[E], q1[E];
    float vx[2][E];
    sm_load_pair<N, E, ST>((const ST *)a.half, (const ST *)a.nyq, r0, t, a0, a1, n0, n1);
    sm_load_line<E, TPL>(p0, p0, 1, true, t, q0);
    sm_load_line<E, TPL>(p1, p1, 1, true, t, q1);
    if constexpr (LOCAL) {
        if (a.bohm) sm_load_pair<N, E, ST>((const ST *)a.half2, (const ST *)a.nyq2, r0, t, b0, b1, m0, m1);
#pragma unroll
        for (int e = 0; e < E; ++e) {
            vx[0][e] = a.vext ? a.vext[r0 * N + t + TPL * e] : 0.0f;
            vx[1][e] = a.vext ? a.vext[r1 * N + t + TPL * e] : 0.0f;
        }
    }
    dc z[1][E], v[2][E];
    sm_join_pair<N, E, ST>(a0, a1, n0, n1, t, z[0]);
    sm_fft<1, N, E, 1, ST>(z, t, lay, lds, 0, tw);
    sm_widen<E>(q0, true, v[0]);
    sm_widen<E>(q1, true, v[1]);
    if constexpr (!REAL_IN) sm_fft<2, N, E, 1, ST>(v, t, lay, lds, STRIDE, tw);
    if constexpr (LOCAL) {
        float lap[2][E];
        dc y[1][E];
        if (a.bohm) {   // uniform over the grid
            sm_join_pair<N, E, ST>(b0, b1, m0, m1, t, y[0]);
            sm_fft<1, N, E, 1, ST>(y, t, lay, lds, 0, tw);
        }
#pragma unroll
        for (int e = 0; e < E; ++e) {
            lap[0][e] = a.bohm ? (float)y[0][e].x : 0.0f;
            lap[1][e] = a.bohm ? (float)y[0][e].y : 0.0f;
        }
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            double rho[E], U[E];
#pragma unroll
            for (int e = 0; e < E; ++e) {
                if constexpr (!REAL_IN) v[b][e] = scl(v[b][e], inv_n);
                rho[e] = norm2(v[b][e]);
            }
            local_potential<E>(a, rho, lap[b], U);
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const double phi = b ? z[0][e].y : z[0][e].x;
                double s, c;
                sincos_tab((U[e] + (double)vx[b][e] + phi) * a.dz, sct, &s, &c);
                v[b][e] = cmul(v[b][e], mk(c, s));
            }
        }
    } else {
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const dc ps = REAL_IN ? v[b][e] : scl(v[b][e], inv_n);
                const double phi = b ? z[0][e].y : z[0][e].x;
                double s, c;
                sincos_tab(fma(a.g, norm2(ps), phi) * a.dz, sct, &s, &c);
                v[b][e] = cmul(ps, mk(c, s));
            }
    }
    sm_fft<2, N, E, -1, ST>(v, t, lay, lds, STRIDE, tw);
    if (act) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            p0[t + TPL * e] = st_c<ST>(v[0][e]);
            p1[t + TPL * e] = st_c<ST>(v[1][e]);
        }
    }
}

// Strided pass (as lm_tile; FWD, INV, KIN and KERN).
template <int N, int LINES, int MODE, class ST>
__device__ __forceinline__ void sm_lm(const LmArgs &a, int tile, double2 *lds)
{
    constexpr int E = SmCfg<N>::E, TPL = N / E;
    static_assert(MODE == LM_FWD || MODE == LM_INV || MODE == LM_KIN || MODE == LM_KERN, "mode");
    const int tid = threadIdx.x, l = tid % LINES, t = tid / LINES;
    const bool second = tile >= a.s0.ntiles;
    const Seg &sg = second ? a.s1 : a.s0;
    if (second) tile -= a.s0.ntiles;
    const int o = tile / sg.ngroups, grp = tile - o * sg.ngroups;
    const int lg = grp * LINES + l;
    const bool act = lg < sg.nlines;
    ST *base = (ST *)sg.ptr + (long long)o * sg.os + (long long)lg * sg.ls;
    const LmLayout<LINES> lay{l};
    ST raw[E];
    dc v[1][E];
    sm_load_line<E, TPL>(base, (const ST *)sg.ptr, sg.es, act, t, raw);
    // inactive lanes (lg >= nlines) read table entry 0, never past the end
    const int c1 = act ? sg.c1f + lg * sg.c1l + o * sg.c1o : 0;
    const int c2 = act ? sg.c2f + lg * sg.c2l + o * sg.c2o : 0;
    dc m12 = mk(0.0, 0.0);
    double q12 = 0.0;
    if constexpr (MODE == LM_KIN) m12 = scl(cmul(from_d2(a.kin1[c1]), from_d2(a.kin2[c2])), a.scale);
    if constexpr (MODE == LM_KERN) q12 = a.k2_1[c1] + a.k2_2[c2];
    sm_widen<E>(raw, act, v[0]);
    sm_fft<1, N, E, MODE == LM_INV ? 1 : -1, ST>(v, t, lay, lds, 0, a.tw);
    if constexpr (MODE == LM_FWD || MODE == LM_INV) {
        if (a.scale != 1.0) {   // uniform
#pragma unroll
            for (int e = 0; e < E; ++e) v[0][e] = scl(v[0][e], a.scale);
        }
    } else {
        if constexpr (MODE == LM_KIN) {
#pragma unroll
            for (int e = 0; e < E; ++e) v[0][e] = cmul(v[0][e], cmul(m12, from_d2(a.kinp[t + TPL * e])));
        } else {
#pragma unroll
            for (int e = 0; e < E; ++e) {
                // branch-free: what k = 0 gives is replaced by 0
                const double k2 = q12 + a.k2_p[t + TPL * e];
                const bool pos = k2 > 0.0;
                const double km = k2 + a.mY2;
                const double num = fma(a.cN, km, a.cY * k2);
                const double den = k2 * km;
                double r = __builtin_amdgcn_rcp(den);
                r = fma(r, fma(-den, r, 1.0), r);
                r = fma(r, fma(-den, r, 1.0), r);
                const double K = pos ? fma(num, r, a.c0) : 0.0;
                v[0][e] = scl(v[0][e], K);
            }
        }
        sm_fft<1, N, E, 1, ST>(v, t, lay, lds, 0, a.tw);
    }
    if (act) {
#pragma unroll
        for (int e = 0; e < E; ++e) base[(long long)(t + TPL * e) * sg.es] = st_c<ST>(v[0][e]);
    }
}

// ---------------------------------------------------------------- kernels
template <int N, int S, class ST = float2>
__global__ __launch_bounds__(SmCfg<N>::WLINES *SmCfg<N>::TPL) void k_sm_em_fft(EmArgs a)
{
    constexpr int LINES = SmCfg<N>::WLINES;
    __shared__ double2 lds[sm_em_slots<N, LINES>() / 2];
    sm_em_fft<N, LINES, S, ST>(a, blockIdx.x, a.tw, lds);
}
template <int N, bool STORE_PSI, class ST = float2>
__global__ __launch_bounds__(SmCfg<N>::WLINES *SmCfg<N>::TPL) void k_sm_density(EmArgs a)
{
    constexpr int LINES = SmCfg<N>::WLINES;
    __shared__ double2 lds[sm_em_slots<N, LINES>()];
    sm_density<N, LINES, STORE_PSI, ST>(a, blockIdx.x, a.tw, lds);
}
template <int N, bool REAL_IN, class ST = float2, bool LOCAL = false>
__global__ __launch_bounds__(SmCfg<N>::WLINES *SmCfg<N>::TPL) void k_sm_phase(EmArgs a)
{
    constexpr int LINES = SmCfg<N>::WLINES;
    __shared__ double2 lds[sm_em_slots<N, LINES>()];
    sm_phase<N, LINES, REAL_IN, LOCAL, ST>(a, blockIdx.x, a.tw, a.sct, lds);
}
// Block ntiles sums the mass partials while the others run the tiles.
template <int N, int MODE, class ST = float2>
__global__ __launch_bounds__(SmCfg<N>::NT) void k_sm_lm(LmArgs a)
{
    constexpr int LINES = SmCfg<N>::LINES;
    __shared__ double2 lds[sm_lm_slots<N, LINES>()];
    if ((int)blockIdx.x == a.s0.ntiles + a.s1.ntiles) {
        __shared__ double sh[SmCfg<N>::NT / 64 + 1];
        if (a.reduce) reduce_mass<SmCfg<N>::NT>(a, sh);
        return;
    }
    sm_lm<N, LINES, MODE, ST>(a, blockIdx.x, lds);
}

}  // namespace gsn
