// gsn_fft.hpp -- device FFT building blocks for gfx950.
//
// A line of N complex points is owned by TPL = N/E threads; thread t holds the
// E points at positions t + TPL*e (e = 0..E-1) in FP64 registers.  The
// transform is a Stockham (self-sorting) mixed-radix DFT: stage s with radix R
// takes butterfly j (t + TPL*m) from positions j + r*N/R, multiplies by the
// twiddles exp(+-2 pi i (j mod Ns) r / (Ns R)), does a length-R DFT in
// registers and sends the outputs to positions expand(j) + r*Ns, with
// expand(j) = (j / Ns) Ns R + (j mod Ns).  Between stages the data goes
// through LDS (complex64 or complex128 slots); the last stage's outputs land in the same
// registers in natural order (position t + TPL*e holds bin t + TPL*e), so a
// pointwise multiplier and an inverse transform can follow without another
// exchange.  Transforms are unnormalised in both directions.
#pragma once
#include <hip/hip_runtime.h>

namespace gsn {

struct dc { double x, y; };

__host__ __device__ __forceinline__ dc mk(double x, double y) { dc r; r.x = x; r.y = y; return r; }
__host__ __device__ __forceinline__ dc add(dc a, dc b) { return mk(a.x + b.x, a.y + b.y); }
__host__ __device__ __forceinline__ dc sub(dc a, dc b) { return mk(a.x - b.x, a.y - b.y); }
__host__ __device__ __forceinline__ dc scl(dc a, double s) { return mk(a.x * s, a.y * s); }
__host__ __device__ __forceinline__ dc conj(dc a) { return mk(a.x, -a.y); }
__host__ __device__ __forceinline__ dc cmul(dc a, dc b)
{
    return mk(fma(a.x, b.x, -a.y * b.y), fma(a.x, b.y, a.y * b.x));
}
__host__ __device__ __forceinline__ double norm2(dc a) { return fma(a.x, a.x, a.y * a.y); }
__device__ __forceinline__ dc from_f2(float2 v) { return mk((double)v.x, (double)v.y); }
__device__ __forceinline__ float2 to_f2(dc v) { return make_float2((float)v.x, (float)v.y); }
__device__ __forceinline__ dc from_d2(double2 v) { return mk(v.x, v.y); }

// LDS exchange slots: complex64 (half the LDS footprint) or complex128 (no
// conversions, no intermediate rounding)
__device__ __forceinline__ void lds_put(float2 *p, int i, dc v) { p[i] = to_f2(v); }
__device__ __forceinline__ void lds_put(double2 *p, int i, dc v) { p[i] = make_double2(v.x, v.y); }
__device__ __forceinline__ dc lds_get(const float2 *p, int i) { return from_f2(p[i]); }
__device__ __forceinline__ dc lds_get(const double2 *p, int i) { return from_d2(p[i]); }

// multiply by S*i (S = -1 forward, +1 inverse)
template <int S> __host__ __device__ __forceinline__ dc mul_si(dc a)
{
    if constexpr (S > 0) return mk(-a.y, a.x);
    else return mk(a.y, -a.x);
}

// cos(pi/8), sin(pi/8), sqrt(1/2)
constexpr double kC1 = 0.92387953251128675613;  // cos(pi/8)
constexpr double kS1 = 0.38268343236508977173;  // sin(pi/8)
constexpr double kR2 = 0.70710678118654752440;  // sqrt(1/2)

// p + w q and p - w q in six FMAs: the difference is 2 p minus the sum.
__host__ __device__ __forceinline__ void bfly(dc &p, dc &q, dc w)
{
    const dc s = mk(fma(w.x, q.x, fma(-w.y, q.y, p.x)), fma(w.x, q.y, fma(w.y, q.x, p.y)));
    q = mk(fma(2.0, p.x, -s.x), fma(2.0, p.y, -s.y));
    p = s;
}
__host__ __device__ __forceinline__ void bfly(dc &p, dc &q)
{
    const dc s = add(p, q);
    q = sub(p, q);
    p = s;
}

// a +- c u (real c)
__host__ __device__ __forceinline__ dc axpy(double c, dc u, dc a) { return mk(fma(c, u.x, a.x), fma(c, u.y, a.y)); }

// DFT4 outputs from the first layer's sums and differences of the points 0, 2
// (s02, d02) and 1, 3 (s13, d13)
template <int S>
__host__ __device__ __forceinline__ void dft4_out(dc s02, dc s13, dc d02, dc d13, dc &x0, dc &x1, dc &x2, dc &x3)
{
    const dc r = mul_si<S>(d13);
    x0 = add(s02, s13);
    x2 = sub(s02, s13);
    x1 = add(d02, r);
    x3 = sub(d02, r);
}

// The same when the points 1 and 3 are c times those of s13 and d13
template <int S>
__host__ __device__ __forceinline__ void dft4_out(double c, dc s02, dc s13, dc d02, dc d13, dc &x0, dc &x1, dc &x2, dc &x3)
{
    const dc r = mul_si<S>(d13);
    x0 = axpy(c, s13, s02);
    x2 = axpy(-c, s13, s02);
    x1 = axpy(c, r, d02);
    x3 = axpy(-c, r, d02);
}

// Length-R DFT in registers, natural order in and out; TW: point r is first
// multiplied by w(r) (r >= 1).  FP64 issue bounds the FFT passes more than memory
// does (a 256-point kinetic pass of 256^3 issues 65 VALU instructions a point, 16.6
// thousand per SIMD: 36 to 45 of its 54 us at the 2.2 to 2.7 ns that an FP64 one
// takes), so the multiplications go into the additions that follow them: a
// twiddled first-layer pair takes 10 instructions instead of 12 (6 instead of 8 for
// point 0), and a constant rotation is applied as c (1, tan) with c folded into the
// next layer's FMAs
// (cos pi/8 or sqrt(1/2); the tangent never exceeds 1).
// FULL: products with twiddles, and with cos and sin of pi/8, are rounded on their
// own.  The short forms err by 1% to 3% more per transform (lines of 16 to 2048
// points against extended precision), the folded pi/8 the same way in every step:
// 12 steps of a complex128 256^2 state on the 16-point plan are 14% further off
// (1.65e-14 against 1.45e-14; shapes with lines up to 1024 points 2% to 14%).
// Beside values that are rounded to complex64 at the next exchange it vanishes, so
// the transforms through complex64 slots, and s4's of complex64 values, are short.
template <int R, int S, bool TW, bool FULL = false, class W>
__host__ __device__ __forceinline__ void dft(dc *a, const W &w)
{
    static_assert(R == 1 || R == 2 || R == 4 || R == 8 || R == 16, "unsupported radix");
    if constexpr (R > 1) {
#pragma unroll
        for (int i = 0; i < R / 2; ++i) {
            if constexpr (TW) {
                if (i > 0) a[i] = cmul(a[i], w(i));
                if constexpr (FULL) {
                    a[i + R / 2] = cmul(a[i + R / 2], w(i + R / 2));
                    bfly(a[i], a[i + R / 2]);
                } else {
                    bfly(a[i], a[i + R / 2], w(i + R / 2));
                }
            } else {
                bfly(a[i], a[i + R / 2]);
            }
        }
    }
    if constexpr (R == 4) {
        dft4_out<S>(a[0], a[1], a[2], a[3], a[0], a[1], a[2], a[3]);
    } else if constexpr (R == 8) {
        // even and odd points, then X[k] = E[k] + w8^k O[k], X[k + 4] = E[k] - w8^k O[k]
        dc e0, e1, e2, e3, o0, o1, o2, o3;
        dft4_out<S>(a[0], a[2], a[4], a[6], e0, e1, e2, e3);
        dft4_out<S>(a[1], a[3], a[5], a[7], o0, o1, o2, o3);
        // w8 = sqrt(1/2) (1 + S i), w8^3 = sqrt(1/2) (-1 + S i)
        const dc r1 = mul_si<S>(o1), r2 = mul_si<S>(o2), r3 = mul_si<S>(o3);
        const dc u1 = add(o1, r1), u3 = sub(r3, o3);
        a[0] = add(e0, o0); a[4] = sub(e0, o0);
        a[1] = axpy(kR2, u1, e1); a[5] = axpy(-kR2, u1, e1);
        a[2] = add(e2, r2); a[6] = sub(e2, r2);
        a[3] = axpy(kR2, u3, e3); a[7] = axpy(-kR2, u3, e3);
    } else if constexpr (R == 16) {
        // 4 x 4: Y_q = DFT4 of the points q, q + 4, q + 8, q + 12;
        // X[k + 4 j] = DFT4 over q of w16^(q k) Y_q[k]
        dc y[4][4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
            dft4_out<S>(a[q], a[q + 4], a[q + 8], a[q + 12], y[q][0], y[q][1], y[q][2], y[q][3]);
        bfly(y[0][0], y[2][0]);
        bfly(y[1][0], y[3][0]);
        dft4_out<S>(y[0][0], y[1][0], y[2][0], y[3][0], a[0], a[4], a[8], a[12]);
        constexpr double t = kS1 / kC1;   // tan(pi/8)
        {   // k = 1: angles pi/8, pi/4, 3 pi/8
            const dc u2 = add(y[2][1], mul_si<S>(y[2][1]));
            const dc p = axpy(kR2, u2, y[0][1]), q = axpy(-kR2, u2, y[0][1]);
            if constexpr (FULL) {
                const dc z1 = cmul(y[1][1], mk(kC1, S * kS1)), z3 = cmul(y[3][1], mk(kS1, S * kC1));
                dft4_out<S>(p, add(z1, z3), q, sub(z1, z3), a[1], a[5], a[9], a[13]);
            } else {
                const dc v = y[1][1], u1 = mk(fma(-S * t, v.y, v.x), fma(S * t, v.x, v.y));
                const dc u3 = mk(fma(t, y[3][1].x, -S * y[3][1].y), fma(t, y[3][1].y, S * y[3][1].x));
                dft4_out<S>(kC1, p, add(u1, u3), q, sub(u1, u3), a[1], a[5], a[9], a[13]);
            }
        }
        {   // k = 2: pi/4, pi/2, 3 pi/4
            const dc u1 = add(y[1][2], mul_si<S>(y[1][2])), u3 = sub(mul_si<S>(y[3][2]), y[3][2]);
            const dc b2 = mul_si<S>(y[2][2]);
            dft4_out<S>(kR2, add(y[0][2], b2), add(u1, u3), sub(y[0][2], b2), sub(u1, u3), a[2], a[6], a[10], a[14]);
        }
        {   // k = 3: 3 pi/8, 3 pi/4, 9 pi/8
            const dc u2 = sub(mul_si<S>(y[2][3]), y[2][3]);
            const dc p = axpy(kR2, u2, y[0][3]), q = axpy(-kR2, u2, y[0][3]);
            if constexpr (FULL) {
                const dc z1 = cmul(y[1][3], mk(kS1, S * kC1)), z3 = cmul(y[3][3], mk(-kC1, -S * kS1));
                dft4_out<S>(p, add(z1, z3), q, sub(z1, z3), a[3], a[7], a[11], a[15]);
            } else {
                const dc u1 = mk(fma(t, y[1][3].x, -S * y[1][3].y), fma(t, y[1][3].y, S * y[1][3].x));
                const dc v = y[3][3], u3 = mk(fma(S * t, v.y, -v.x), fma(-S * t, v.x, -v.y));
                dft4_out<S>(kC1, p, add(u1, u3), q, sub(u1, u3), a[3], a[7], a[11], a[15]);
            }
        }
    }
}

// Stage plan: ceil(log_E N) stages, the first of radix N / E^(stages - 1)
// (the smallest), the others of radix E.  The short radix goes first because
// a short last stage, combining two halves that were just rounded to
// complex64 in the LDS exchange, biases the norm over long runs: 2000 steps
// of the 8-lump 512^3 state drift by -2.8e-6 with radices 16,16,2 and by
// -6.5e-8 with 2,16,16; 2000 steps at 128^3 by -8.8e-7 with 8,8,2 and by
// 3.8e-8 with 2,8,8.
template <int N, int E> struct Plan {
    static_assert(N >= E && N % E == 0, "E must divide N");
    static constexpr int TPL = N / E;
    static constexpr int nstages()
    {
        int s = 0;
        long p = 1;
        while (p < N) { p *= E; ++s; }
        return s;
    }
    static constexpr int radix(int s)
    {
        if (s > 0) return E;
        int r = N;
        for (int i = 1; i < nstages(); ++i) r /= E;
        return r;
    }
    static constexpr int ns(int s)
    {
        int p = 1;
        for (int i = 0; i < s; ++i) p *= radix(i);
        return p;
    }
};

// LDS addressing of one line.  Element-major lines (contiguous axis): one pad
// per 16 points plus a line pitch of 16 (mod 32) float2.  Line-major tiles
// (strided axes): position-major with the LINES lines of a tile adjacent.
// Synchronisation of an LDS exchange: a block barrier, or (when every line of
// the tile lives inside one wavefront) a wavefront-scope fence plus a wave
// barrier, which orders the wave's own LDS writes before its reads.
template <bool WAVE> __device__ __forceinline__ void exchange_sync()
{
    if constexpr (WAVE) {
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    } else {
        __syncthreads();
    }
}

template <int N, int E = 16> struct EmLayout {
    // one pad slot per E points: the first-stage writes (E consecutive
    // positions per lane) then hit distinct banks across a wavefront
    static constexpr int PAD_SHIFT = E >= 16 ? 4 : E == 8 ? 3 : E == 4 ? 2 : 1;
    static constexpr int S0 = N + (N >> PAD_SHIFT);
    static constexpr int PITCH = (S0 % 32 == 0) ? S0 + 16 : S0;
    static constexpr int BYTES_PER_LINE = PITCH * 8;
    static constexpr bool WAVE_LOCAL = (N / E) <= 64;   // a row within one wavefront
    int base;
    __device__ __forceinline__ int operator()(int pos) const { return base + pos + (pos >> PAD_SHIFT); }
};
template <int LINES> struct LmLayout {
    static constexpr bool WAVE_LOCAL = false;
    int l;
    __device__ __forceinline__ int operator()(int pos) const { return pos * LINES + l; }
};

// The twiddles of butterfly jm of a stage: w(r) = exp(S 2 pi i jm r STEP / N).
template <int STEP, int S> struct Twiddles {
    const double2 *__restrict__ tw;
    int jm;
    __device__ __forceinline__ dc operator()(int r) const
    {
        const double2 w = tw[jm * r * STEP];
        return mk(w.x, S > 0 ? -w.y : w.y);
    }
};

// Whether a transform with LT exchange slots computes to full FP64 accuracy.
template <class LT> constexpr bool kFullFp64 = sizeof(LT) == sizeof(double2);

// One Stockham stage and the recursion over the remaining stages.
template <int N, int E, int S, int ST, class Lay, class LT>
__device__ __forceinline__ void fft_stages(dc (&v)[E], int t, const Lay &lay, LT *lds,
                                           const double2 *__restrict__ tw)
{
    using P = Plan<N, E>;
    if constexpr (ST < P::nstages()) {
        constexpr int R = P::radix(ST);
        constexpr int NS = P::ns(ST);
        constexpr bool LAST = (ST + 1 == P::nstages());
        constexpr int B = E / R;
        constexpr int TPL = P::TPL;
#pragma unroll
        for (int m = 0; m < B; ++m) {
            const int j = t + TPL * m;
            dc a[R];
#pragma unroll
            for (int r = 0; r < R; ++r) a[r] = v[m + r * B];
            dft<R, S, (NS > 1), kFullFp64<LT>>(a, Twiddles<N / (NS * R), S>{tw, j & (NS - 1)});
            if constexpr (LAST) {
#pragma unroll
                for (int r = 0; r < R; ++r) v[m + r * B] = a[r];
            } else {
                const int base = (j / NS) * NS * R + (j & (NS - 1));
#pragma unroll
                for (int r = 0; r < R; ++r) lds_put(lds, lay(base + r * NS), a[r]);
            }
        }
        if constexpr (!LAST) {
            exchange_sync<Lay::WAVE_LOCAL>();
#pragma unroll
            for (int e = 0; e < E; ++e) v[e] = lds_get(lds, lay(t + TPL * e));
            exchange_sync<Lay::WAVE_LOCAL>();
            fft_stages<N, E, S, ST + 1>(v, t, lay, lds, tw);
        }
    }
}

// Unnormalised DFT of the line held in v (S = -1 forward, +1 inverse).
// tw[q] = exp(-2 pi i q / N), q < N, FP64 (global or LDS).  Every thread of the block must
// call this (it contains barriers when the plan has more than one stage).
template <int N, int E, int S, class Lay, class LT>
__device__ __forceinline__ void fft(dc (&v)[E], int t, const Lay &lay, LT *lds,
                                    const double2 *__restrict__ tw)
{
    fft_stages<N, E, S, 0>(v, t, lay, lds, tw);
}

// Deterministic FP64 block sum (result valid in thread 0).
template <int NT> __device__ __forceinline__ double block_sum(double v, double *sh)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    const int tid = threadIdx.x;
    if constexpr (NT > 64) {
        if ((tid & 63) == 0) sh[tid >> 6] = v;
        __syncthreads();
        if (tid == 0) {
            double s = 0.0;
#pragma unroll
            for (int w = 0; w < NT / 64; ++w) s += sh[w];
            v = s;
        }
        __syncthreads();
    }
    return v;
}

}  // namespace gsn
