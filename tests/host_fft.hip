// Host build of the FFT butterflies (the same inline functions the passes run on
// the GPU): the error of forward transforms of lines against extended precision,
// with the butterflies of a complex128 exchange, and with every product with a
// twiddle rounded before it is added and subtracted, on the same stage plan.
// Prints N, E, the kind of line, and both relative errors.
#include <cmath>
#include <complex>
#include <cstdio>
#include <random>
#include <vector>
#include "gsn_fft.hpp"

using gsn::dc;
using gsn::mk;
typedef std::complex<long double> ld;

static std::vector<double2> g_tw;
constexpr bool kFull = gsn::kFullFp64<double2>;

template <int N, int E, int ST, bool PRODUCTS> static void stages(std::vector<dc> &v)
{
    using P = gsn::Plan<N, E>;
    if constexpr (ST < P::nstages()) {
        constexpr int R = P::radix(ST), NS = P::ns(ST);
        std::vector<dc> o(N);
        for (int j = 0; j < N / R; ++j) {
            const int jm = j & (NS - 1);
            auto w = [&](int r) { return mk(g_tw[jm * r * (N / (NS * R))].x, g_tw[jm * r * (N / (NS * R))].y); };
            dc a[R];
            for (int r = 0; r < R; ++r) a[r] = v[j + r * (N / R)];
            if constexpr (PRODUCTS) {
                for (int r = 1; r < R; ++r) a[r] = gsn::cmul(a[r], w(r));
                gsn::dft<R, -1, false, kFull>(a, w);
            } else {
                gsn::dft<R, -1, (NS > 1), kFull>(a, w);
            }
            for (int r = 0; r < R; ++r) o[(j / NS) * NS * R + jm + r * NS] = a[r];
        }
        v = o;
        stages<N, E, ST + 1, PRODUCTS>(v);
    }
}

static void exact(std::vector<ld> &x)
{
    const int n = (int)x.size();
    if (n == 1) return;
    std::vector<ld> a(n / 2), b(n / 2);
    for (int i = 0; i < n / 2; ++i) { a[i] = x[2 * i]; b[i] = x[2 * i + 1]; }
    exact(a);
    exact(b);
    for (int k = 0; k < n / 2; ++k) {
        const long double t = -2.0L * 3.14159265358979323846264338327950288L * k / n;
        const ld u = ld(cosl(t), sinl(t)) * b[k];
        x[k] = a[k] + u;
        x[k + n / 2] = a[k] - u;
    }
}

template <int N, int E> static void run()
{
    g_tw.resize(N);
    for (int q = 0; q < N; ++q) {
        const double t = 2.0 * M_PI * q / N;
        g_tw[q] = make_double2(std::cos(t), -std::sin(t));
    }
    for (int smooth = 0; smooth < 2; ++smooth) {
        std::mt19937_64 gen(5);
        std::normal_distribution<double> nd;
        long double e = 0, et = 0, norm = 0;
        for (int it = 0; it < (1 << 17) / N; ++it) {
            const double c = nd(gen), k = 3.0 * nd(gen);
            std::vector<ld> y(N);
            std::vector<dc> x(N), xt;
            for (int i = 0; i < N; ++i) {
                const double u = (i - N / 2.0) / (N / 8.0) + c, env = std::exp(-u * u);
                x[i] = smooth ? mk(env * std::cos(k * u), env * std::sin(k * u)) : mk(nd(gen), nd(gen));
                y[i] = ld(x[i].x, x[i].y);
            }
            xt = x;
            exact(y);
            stages<N, E, 0, false>(x);
            stages<N, E, 0, true>(xt);
            for (int i = 0; i < N; ++i) {
                norm += std::norm(y[i]);
                e += std::norm(ld(x[i].x, x[i].y) - y[i]);
                et += std::norm(ld(xt[i].x, xt[i].y) - y[i]);
            }
        }
        std::printf("%d %d %d %.6e %.6e\n", N, E, smooth, (double)sqrtl(e / norm), (double)sqrtl(et / norm));
    }
}

template <int N> static void plans() { run<N, 16>(); run<N, 8>(); run<N, 4>(); }

int main()
{
    plans<16>();
    plans<64>();
    plans<128>();
    plans<256>();
    plans<512>();
    plans<1024>();
    plans<2048>();
    return 0;
}
