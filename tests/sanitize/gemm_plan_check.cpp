// Scratch bounds of the contractions against the plans they have to cover:
// prints "ok <plans>" or the first plan that needs more than its bound.
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <random>

#include "../../paper_1812_01329_amd/csrc/gemm_plan.hpp"

using namespace janus;

static size_t need(const GemmDesc& g) {
    if (g.dtype == JANUS_F32) {
        const int n = f32_splits(g);
        return n > 1 ? size_t(n) * g.M * g.N * 4 : 0;
    }
    const NtPlan p = plan_nt(g);
    return p.fast ? p.bytes : 0;
}

static long plans = 0;
static void check(GemmDesc g, GemmSize size, int step) {
    const size_t bound = gemm_scratch_bound(g, size);
    const int top = size == GemmSize::kUpToM ? g.M : size == GemmSize::kUpToK ? g.K : 1;
    for (int v = top; v >= 1; v -= step) {
        GemmDesc q = g;
        if (size == GemmSize::kUpToM) q.M = v;
        if (size == GemmSize::kUpToK) q.K = v;
        ++plans;
        if (need(q) > bound) {
            std::printf("dtype %d layout %d%d: %d x %d over %d needs %zu bytes, bound %zu (of %d x %d over %d, size %d)\n",
                        int(g.dtype), int(g.a_t), int(g.b_t), q.M, q.N, q.K, need(q), bound, g.M, g.N, g.K, int(size));
            std::exit(1);
        }
    }
}

int main() {
    std::mt19937 rng(17);
    auto draw = [&](int lo, int hi) {   // even over the logarithm
        const double u = std::uniform_real_distribution<double>(0.0, 1.0)(rng);
        return int(lo * std::pow(double(hi) / lo, u) + 0.5);
    };
    for (janus_dtype dt : {JANUS_BF16, JANUS_F32}) {
        GemmDesc w;   // a weight gradient: K = running rows of a ragged batch
        w.dtype = dt;
        w.a_zero_pad = true;
        w.b_t = true;
        const int cases[][3] = {{320, 240, 2160}, {480, 120, 4536}, {480, 240, 4536}, {16, 16, 70000}, {2624, 656, 5000}};
        for (const auto& c : cases) {
            w.M = c[0];
            w.N = c[1];
            w.K = c[2];
            check(w, GemmSize::kUpToK, 1);
        }
        for (int i = 0; i < 3000; ++i) {
            w.M = draw(1, 9000);
            w.N = draw(1, 3000);
            w.K = draw(1, 30000);
            w.a_t = i % 3 == 2;
            w.a_zero_pad = !w.a_t;
            check(w, GemmSize::kUpToK, std::max(1, w.K / 200));
            GemmDesc x;   // an input projection, or the gradient of an input: M = running rows
            x.dtype = dt;
            x.M = draw(1, 70000);
            x.N = draw(1, 9000);
            x.K = draw(1, 5000);
            x.b_t = i % 2 == 1;
            check(x, GemmSize::kUpToM, std::max(1, x.M / 200));
            check(x, GemmSize::kExact, 1);
        }
    }
    std::printf("ok %ld\n", plans);
    return 0;
}
