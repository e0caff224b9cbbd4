// FP16 storage: the half step sums <r~, s> over s as it is stored, and p takes
// up r as it is stored (r and rho are formed from those).  ||s||^2 and ||r||^2
// are over the values before storage.
#include "block_emu.hpp"

#include "blas.hip"

#include <random>

static constexpr int kVh = 96;
static std::mt19937 rng(11);
static float gauss() { return std::normal_distribution<float>()(rng); }

int main() {
    std::vector<std::vector<char>> v;  // r, q, r~, p, t, (x in FP32)
    for (int k = 0; k < 5; k++) {
        v.emplace_back(spinor_bytes(P16, kVh));
        for (int i = 0; i < kVh; i++) {
            Spinor<float> s;
            for (auto &c : s.c) c = {gauss(), gauss()};
            SpinorIO<P16>::store(v[k].data(), kVh, i, s);
        }
    }
    std::vector<char> x(spinor_bytes(P32, kVh), 0);
    std::vector<double> sc(S_COUNT, 0.0), parts(3 * 2, 0.0), in0(5), in1(3);
    std::vector<int> fl(F_COUNT, 0);
    VecBatch B;
    std::memset(&B, 0, sizeof(B));
    B.h.S = 1;
    B.h.off[1] = 2;
    VecCall &c = B.c[0];
    c.Vh = kVh;
    c.sc = sc.data();
    c.fl = fl.data();
    c.partials = parts.data();
    c.in0 = SumSource{in0.data(), 1};
    c.in1 = SumSource{in1.data(), 1};
    c.guard = 1;
    int bad = 0;

    sc[S_RHO0] = 0.3;
    in0 = {0.5, 0.1, 0, 0, 0};
    c.a = v[0].data(), c.b = v[1].data(), c.c = v[2].data();
    for (int b = 0; b < 2; b++) emu::run_block(b, 2, 64, [&] { k_vec<V_INNER_A, P16, P32>(B); });
    {
        double re = 0, im = 0, size = 0, ss = 0;
        for (int i = 0; i < kVh; i++) {
            const Spinor<float> a = SpinorIO<P16>::load(v[2].data(), kVh, i), s = SpinorIO<P16>::load(v[0].data(), kVh, i);
            for (int k = 0; k < 12; k++) {
                const double ar = a.c[k].re, ai = a.c[k].im, sr = s.c[k].re, si = s.c[k].im;
                re += ar * sr + ai * si;
                im += ar * si - ai * sr;
                ss += sr * sr + si * si;
                size += std::sqrt((ar * ar + ai * ai) * (sr * sr + si * si));
            }
        }
        const double er = std::hypot(parts[2] + parts[3] - re, parts[4] + parts[5] - im);
        if (er > 1e-12 * size) {
            std::printf("half step: <r~, s> off by %.3g of %.3g\n", er, size);
            bad++;
        }
        if (std::fabs(parts[0] + parts[1] - ss) > 2e-3 * ss) {
            std::printf("half step: ||s||^2\n");
            bad++;
        }
    }

    // p = r + beta (p - omega q)
    in0 = {0.2, 0.1, 2.0, 0.1, 0.05};
    in1 = {1.0, 0.1, 0.02};
    const cx<double> rho = {sc[S_RHO1], sc[S_RHO1 + 1]}, al = cdiv(rho, {sc[S_RQ], sc[S_RQ + 1]});
    const cx<double> om = {in0[0] / in0[2], -in0[1] / in0[2]};
    const cx<double> rho1 = cx<double>{in1[1], in1[2]} - om * cx<double>{in0[3], in0[4]};
    const cx<double> beta = cdiv(rho1, rho) * cdiv(al, om);
    const auto p0 = v[3];
    c.a = x.data(), c.b = v[0].data(), c.c = v[3].data(), c.d = v[4].data(), c.e = v[1].data();
    for (int b = 0; b < 2; b++) emu::run_block(b, 2, 64, [&] { k_vec<V_INNER_B, P16, P32>(B); });
    double worst = 0;
    for (int i = 0; i < kVh; i++) {
        const Spinor<float> r = SpinorIO<P16>::load(v[0].data(), kVh, i), q = SpinorIO<P16>::load(v[1].data(), kVh, i),
                            p = SpinorIO<P16>::load(v[3].data(), kVh, i), o = SpinorIO<P16>::load(p0.data(), kVh, i);
        const double m = *tp<float, 52>(v[3].data(), i, 48);
        for (int k = 0; k < 12; k++) {
            const cx<double> qk = {q.c[k].re, q.c[k].im}, ok = {o.c[k].re, o.c[k].im};
            const cx<double> w = cx<double>{r.c[k].re, r.c[k].im} + beta * (ok - om * qk);
            worst = std::max(worst, std::max(std::fabs(p.c[k].re - w.re), std::fabs(p.c[k].im - w.im)) / m);
        }
    }
    // its own storage rounding alone: half a unit of a half below 1, and FP32 arithmetic
    if (worst > std::ldexp(1.0, -12) + 1e-5) {
        std::printf("closing update: p is off by %.3g of its scale\n", worst);
        bad++;
    }
    if (bad) return 1;
    std::printf("ok\n");
    return 0;
}
