// The inner loop's updates stop as whole blocks.  An update that finds the loop
// converged raises a done code while other blocks of its own launch are under
// way; here block 0 does so while another block's first wavefront waits at the
// barrier of its sums and the second has not started.  Whatever that wavefront
// reads, the block must leave every vector alone, and so must the next update.
// The LDS holds the sums of an earlier launch, far above the tolerance.
#include "block_emu.hpp"

#include "blas.hip"

#include <random>
#include <thread>

static constexpr int kVh = 200, kBs = 128, kNblk = 2, kParts = 128;

struct Sys {
    std::vector<std::vector<char>> v;
    std::vector<double> sc, parts, in0, in1;
    std::vector<int> fl;
    Sys(unsigned seed, int nvec) : sc(S_COUNT, 0.0), parts(8 * kNblk, 0.0), in0(5 * kParts, 0.0), in1(3 * kParts, 0.0), fl(F_COUNT, 0) {
        std::mt19937 r(seed);
        std::normal_distribution<double> g;
        for (int k = 0; k < nvec; k++) {
            v.emplace_back(spinor_bytes(P64, kVh));
            double *d = (double *)v.back().data();
            for (size_t j = 0; j < v.back().size() / 8; j++) d[j] = g(r);
        }
    }
    void sums(std::vector<double> &in, std::initializer_list<double> tot) {
        int k = 0;
        for (double t : tot) {
            for (int j = 0; j < kParts; j++) in[k * kParts + j] = t / kParts;
            k++;
        }
    }
    VecBatch batch(std::initializer_list<int> order) {
        VecBatch B;
        std::memset(&B, 0, sizeof(B));
        B.h.S = 1;
        B.h.off[1] = kNblk;
        VecCall &c = B.c[0];
        void **f[] = {&c.a, &c.b, &c.c, &c.d, &c.e};
        int k = 0;
        for (int o : order) *f[k++] = v[o].data();
        c.Vh = kVh;
        c.sc = sc.data();
        c.fl = fl.data();
        c.partials = parts.data();
        c.in0 = SumSource{in0.data(), kParts};
        c.in1 = SumSource{in1.data(), kParts};
        c.guard = 1;
        c.bs = kBs;
        return B;
    }
};

template <int OP> void launch(const VecBatch &B) {
    for (int b = 0; b < kNblk; b++) emu::run_block(b, kNblk, kBs, [&] { k_vec<OP, P64, P64>(B); });
}
// block 0 runs while block 1 is between its wavefronts
template <int OP> void launch_interleaved(const VecBatch &B) {
    emu::run_block(1, kNblk, kBs, [&] { k_vec<OP, P64, P64>(B); }, [&](int w) {
        if (w != 0) return;
        std::thread([&] { emu::run_block(0, kNblk, kBs, [&] { k_vec<OP, P64, P64>(B); }); }).join();
    });
}

// r 0, q 1, r~ 2, p 3, t 4, x 5
static const std::initializer_list<int> kA = {0, 1, 2}, kB = {5, 0, 3, 4, 1};

static int expect(const char *what, bool ok) {
    if (!ok) std::printf("%s\n", what);
    return ok ? 0 : 1;
}

int main() {
    int bad = 0;
    {  // the full-step stop, found by the half-step update
        Sys before(1, 6), s(2, 6);
        before.fl[F_ITERS] = s.fl[F_ITERS] = 3;
        before.sc[S_TOL2] = s.sc[S_TOL2] = 1e-6;
        before.sc[S_RHO0] = s.sc[S_RHO0] = 0.3;
        before.sums(before.in0, {0.5, 0.1});
        before.sums(before.in1, {10.0});
        s.sums(s.in0, {0.5, 0.1});
        s.sums(s.in1, {1e-9});
        launch<V_INNER_A>(before.batch(kA));
        const auto v0 = s.v;
        launch_interleaved<V_INNER_A>(s.batch(kA));
        bad += expect("half-step update: vectors changed after a stop", s.v == v0);
        s.sums(s.in0, {0.2, 0.1, 2.0, 0.1, 0.1});
        s.sums(s.in1, {1.0, 0.1, 0.1});
        launch<V_INNER_B>(s.batch(kB));
        bad += expect("the update after a stop changed vectors", s.v == v0);
        bad += expect("the done code is lost", s.fl[F_DONE] == DONE_FULL && s.fl[F_ITERS] == 3);
        launch<V_INNER_A>(s.batch(kA));
        launch<V_INNER_B>(s.batch(kB));
        bad += expect("a later iteration changed vectors", s.v == v0 && s.fl[F_DONE] == DONE_FULL);
    }
    {  // the half-step stop, found by the closing update
        Sys before(3, 6), s(4, 6);
        for (Sys *q : {&before, &s}) {
            q->sc[S_TOL2] = 1e-6;
            q->sc[S_RHO1] = 0.3;
            q->sc[S_RQ] = 0.5;
            q->sums(q->in0, {0.2, 0.1, 2.0, 0.1, 0.1});
        }
        before.sums(before.in1, {10.0, 0.1, 0.1});
        s.sums(s.in1, {1e-9, 0.1, 0.1});
        launch<V_INNER_B>(before.batch(kB));
        const auto v0 = s.v;
        launch_interleaved<V_INNER_B>(s.batch(kB));
        bad += expect("closing update: vectors changed after a stop", s.v == v0);
        bad += expect("the half-step stop is not recorded", s.fl[F_DONE] == DONE_HALF && s.fl[F_ITERS] == 0);
        launch<V_INNER_A>(s.batch(kA));
        launch<V_INNER_B>(s.batch(kB));
        bad += expect("a later iteration changed vectors", s.v == v0 && s.fl[F_DONE] == DONE_HALF);
    }
    if (bad) return 1;
    std::printf("ok\n");
    return 0;
}
