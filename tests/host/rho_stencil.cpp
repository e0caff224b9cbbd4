// FP16 storage: the D-hat halves of the inner loop sum <r~, t> over t as it is
// stored, since r is formed from the stored t and rho is <r~, r>.  The sums
// <s, t> and ||t||^2 that omega is made of are over the values before storage.
// Every kernel that a launch may take, on a ragged lattice.
#include "block_emu.hpp"

#include "dslash.hip"

#include <random>

static Geom geom() {
    Geom g;
    g.L[0] = 6, g.L[1] = 4, g.L[2] = 4, g.L[3] = 2;
    g.Lxh = 3;
    g.Vh = 96;  // one tile and a half
    return g;
}

static std::mt19937 rng(7);
static float gauss() { return std::normal_distribution<float>()(rng); }

static std::vector<char> spinors(int Vh) {
    std::vector<char> v(spinor_bytes(P16, Vh));
    for (int i = 0; i < Vh; i++) {
        Spinor<float> s;
        for (auto &c : s.c) c = {gauss(), gauss()};
        SpinorIO<P16>::store(v.data(), Vh, i, s);
    }
    return v;
}
static std::vector<char> halves(size_t bytes, float size) {
    std::vector<char> v(bytes);
    uint32_t *u = (uint32_t *)v.data();
    for (size_t k = 0; k < bytes / 4; k++) u[k] = f2h(size * gauss(), size * gauss());
    return v;
}

struct Dot {
    double re = 0, im = 0, size = 0;
    void add(cx<double> a, cx<double> b) {
        re += a.re * b.re + a.im * b.im;
        im += a.re * b.im - a.im * b.re;
        size += std::sqrt((a.re * a.re + a.im * a.im) * (b.re * b.re + b.im * b.im));
    }
};
// <a, b> over stored fields
static Dot dot(const std::vector<char> &a, const std::vector<char> &b, int Vh) {
    Dot d;
    for (int i = 0; i < Vh; i++) {
        const Spinor<float> x = SpinorIO<P16>::load(a.data(), Vh, i), y = SpinorIO<P16>::load(b.data(), Vh, i);
        for (int k = 0; k < 12; k++) d.add({x.c[k].re, x.c[k].im}, {y.c[k].re, y.c[k].im});
    }
    return d;
}

static const int kSys = 3;
struct Fields {
    Geom g = geom();
    std::vector<char> links, clov, in[kSys], cen[kSys], rt[kSys], out[kSys];
    std::vector<double> part[kSys];
    Fields() {
        links = halves(8 * link_slab_bytes(P16, g.Vh), 0.4f);
        clov = halves(clover_slab_bytes(P16, g.Vh), 0.3f);
        for (int i = 0; i < g.Vh; i++) *(float *)tp<float, 148>(clov.data(), i, 144) = 1.0f;
        for (int s = 0; s < kSys; s++) {
            in[s] = spinors(g.Vh);
            cen[s] = spinors(g.Vh);
            rt[s] = spinors(g.Vh);
            out[s].assign(spinor_bytes(P16, g.Vh), 0);
            part[s].assign(5 * 2, 0.0);
        }
    }
    MultBatch one(int nblk) {
        MultBatch B;
        std::memset(&B, 0, sizeof(B));
        B.h.S = 1;
        B.h.off[1] = nblk;
        MultKArgs &a = B.d[0];
        a.g = g;
        a.out = out[0].data();
        a.in = in[0].data();
        a.center = cen[0].data();
        a.aux = rt[0].data();
        a.links = links.data();
        a.link_slab = link_slab_bytes(P16, g.Vh);
        a.clov = clov.data();
        a.coef = -0.02;
        a.red.partials = part[0].data();
        a.nblk = nblk;
        return B;
    }
    MrhsArgs all(int ngroups) {
        MrhsArgs A;
        std::memset(&A, 0, sizeof(A));
        A.g = g;
        A.links = links.data();
        A.link_slab = link_slab_bytes(P16, g.Vh);
        A.clov = clov.data();
        A.coef = -0.02;
        A.nsys = kSys;
        A.ngroups = ngroups;
        A.ntiles = 2;
        for (int s = 0; s < kSys; s++)
            A.s[s] = MrhsSys{out[s].data(), in[s].data(), cen[s].data(), rt[s].data(), part[s].data(), nullptr};
        return A;
    }
    // [<s,t>, ||t||^2, <r~,t>], each with nblk partials
    int check(const char *name, int s, int nblk) {
        double v[5] = {0, 0, 0, 0, 0};
        for (int k = 0; k < 5; k++)
            for (int j = 0; j < nblk; j++) v[k] += part[s][k * nblk + j];
        const Dot st = dot(cen[s], out[s], g.Vh), tt = dot(out[s], out[s], g.Vh), rt_t = dot(rt[s], out[s], g.Vh);
        int bad = 0;
        // FP64 sums of the same products in another order
        if (std::hypot(v[3] - rt_t.re, v[4] - rt_t.im) > 1e-12 * rt_t.size) bad = 1;
        // before and after storage: half a unit in the last place of a half, per
        // entry and relative to the site's largest
        if (std::hypot(v[0] - st.re, v[1] - st.im) > 2e-3 * st.size || std::fabs(v[2] - tt.re) > 2e-3 * tt.re) bad |= 2;
        if (bad) std::printf("%s system %d: wrong sums %d, <r~,t> off by %.3g of %.3g\n", name, s, bad,
                             std::hypot(v[3] - rt_t.re, v[4] - rt_t.im), rt_t.size);
        return bad != 0;
    }
};

int main() {
    int bad = 0;
    {
        Fields f;
        const MultBatch B = f.one(2);
        for (int b = 0; b < 2; b++) emu::run_block(b, 2, 256, [&] { k_mult_split<P16, M_DHAT, R_STEP, STREAM, 12>(B); });
        bad += f.check("k_mult_split", 0, 2);
    }
    {
        Fields f;
        const MultBatch B = f.one(2);
        for (int b = 0; b < 2; b++) emu::run_block(b, 2, 64, [&] { k_mult<P16, M_DHAT, R_STEP, SHARED, 12>(B); });
        bad += f.check("k_mult", 0, 2);
    }
    {
        Fields f;
        const MrhsArgs A = f.all(1);
        for (int b = 0; b < 2; b++) emu::run_block(b, 2, 128, [&] { k_mult_multi<P16, M_DHAT, R_STEP, 12>(A); });
        for (int s = 0; s < kSys; s++) bad += f.check("k_mult_multi", s, 2);
    }
    {
        Fields f;
        const MrhsArgs A = f.all(2);
        for (int b = 0; b < 2; b++) emu::run_block(b, 2, 128, [&] { k_mult_mrhs<P16, M_DHAT, R_STEP, 12, 2>(A); });
        for (int s = 0; s < kSys; s++) bad += f.check("k_mult_mrhs", s, 2);
    }
    if (bad) return 1;
    std::printf("ok\n");
    return 0;
}
