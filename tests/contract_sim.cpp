// Replays the operand loads of the contraction kernels on the CPU: for random
// contractions and every tile shape, the bytes that each lane of each tile and
// step reads, with the planner's offsets and the kernel's own address
// formation, have to lie inside the operand.  contract_sim SEED COUNT
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "contract_kernel.h"
#include "ttx_internal.h"

using namespace ttx;

namespace ttx {
hipError_t launch_contract_f32(const ContractPlan&, const float*, const float*, float*, float*, float, float,
                               hipStream_t) {
    return hipSuccess;
}
hipError_t launch_contract_f64(const ContractPlan&, const double*, const double*, double*, double*, double, double,
                               hipStream_t) {
    return hipSuccess;
}
}  // namespace ttx

static const char* const kBase = reinterpret_cast<const char*>(uintptr_t(1) << 40);
static int64_t replayed[2];   // units loaded by lanes within the walk, and beyond it

// One operand's loads for one tile and step.
template <typename T, int ROWS, int KT, bool KW, bool VEC>
static bool step_in_bounds(const int64_t* rows, const int64_t* koff, int wa, int wb, int used, int64_t bytes) {
    using Load = ContractLoad<T, ROWS, KT, KW, VEC>;
    for (int tid = 0; tid < 256; ++tid) {
        Load l;
        l.init(tid, reinterpret_cast<const T*>(kBase), rows, wa, wb, used);
        ++replayed[tid % Load::P >= Load::W];
        for (int i = 0; i < Load::N; ++i)
            for (int j = 0; j < (VEC ? 1 : Load::U); ++j) {
                const int64_t at = l.from(koff, i, j) - kBase;
                if (at < 0 || at + int64_t(VEC ? 16 : sizeof(T)) > bytes) return false;
            }
    }
    return true;
}

template <typename T, int MB, int NB, bool XK, bool YK, bool VEC>
static bool loads_in_bounds(const ContractPlan& p, int64_t bytes_x, int64_t bytes_y) {
    constexpr int MT = 64 * MB, NT = 16 * NB, KT = contract_kt(sizeof(T), MB);
    const ContractArgs& a = p.args;
    auto tables = [](const ContractGroup& g, int64_t first, int n, int used, std::vector<int64_t>* o0,
                     std::vector<int64_t>* o1) {
        o0->assign(n, 0);
        o1->assign(n, 0);
        for (int r = 0; r < n; ++r) {
            int64_t x, y;
            if (r >= used || !g.offsets(first + r, &x, &y)) continue;
            (*o0)[r] = x * int64_t(sizeof(T));
            (*o1)[r] = y * int64_t(sizeof(T));
        }
    };
    std::vector<int64_t> rows, unused, kx, ky;
    for (int64_t s = 0; s < a.steps; ++s) {
        tables(a.k, s * KT, KT, KT, &kx, &ky);
        for (int64_t t = 0; t < a.tiles_m; ++t) {
            tables(a.m, t * a.rows, MT, a.rows, &rows, &unused);
            if (!step_in_bounds<T, MT, KT, XK, VEC>(rows.data(), kx.data(), XK ? 1 : a.walk_x, a.walk_y, a.rows, bytes_x))
                return false;
        }
        for (int64_t t = 0; t < a.tiles_n; ++t) {
            tables(a.n, t * NT, NT, NT, &rows, &unused);
            if (!step_in_bounds<T, NT, KT, YK, VEC>(rows.data(), ky.data(), XK && YK && a.kwalk_x > 1 ? a.kwalk_y : 1,
                                                    a.kwalk_x, KT, bytes_y))
                return false;
        }
    }
    return true;
}

template <typename T, int MB, int NB>
static bool tile_in_bounds(const ContractPlan& p, int64_t bx, int64_t by) {
    const int form = (p.xk ? 4 : 0) + (p.yk ? 2 : 0) + (p.vec_xy ? 1 : 0);
    switch (form) {
        case 0: return loads_in_bounds<T, MB, NB, false, false, false>(p, bx, by);
        case 1: return loads_in_bounds<T, MB, NB, false, false, true>(p, bx, by);
        case 2: return loads_in_bounds<T, MB, NB, false, true, false>(p, bx, by);
        case 3: return loads_in_bounds<T, MB, NB, false, true, true>(p, bx, by);
        case 4: return loads_in_bounds<T, MB, NB, true, false, false>(p, bx, by);
        case 5: return loads_in_bounds<T, MB, NB, true, false, true>(p, bx, by);
        case 6: return loads_in_bounds<T, MB, NB, true, true, false>(p, bx, by);
        default: return loads_in_bounds<T, MB, NB, true, true, true>(p, bx, by);
    }
}

template <typename T>
static bool in_bounds(const ContractPlan& p, int64_t bx, int64_t by) {
    switch (p.variant) {
#define TTX_CASE(i, mb, nb) \
    case i: return tile_in_bounds<T, mb, nb>(p, bx, by);
        TTX_CONTRACT_MENU(TTX_CASE)
#undef TTX_CASE
        default: return false;
    }
}

int main(int argc, char** argv) {
    std::mt19937 r(argc > 1 ? std::atoi(argv[1]) : 0);
    const int count = argc > 2 ? std::atoi(argv[2]) : 100;
    auto draw = [&](int lo, int hi) { return int(r() % uint32_t(hi - lo + 1)) + lo; };
    int vec = 0, wide = 0;
    for (int it = 0; it < count; ++it) {
        // rows, columns and the sum: one to three labels each; every other time
        // the first label of each group is a multiple of 16
        const int nm = draw(1, 3), nn = draw(1, 3), nk = draw(1, 3), c = nm + nn + nk;
        std::vector<ContractLabel> L(c);
        std::vector<int> order[3];
        for (int i = 0; i < c; ++i) {
            const bool first = i == 0 || i == nm || i == nm + nn;
            L[i] = ContractLabel{!first ? draw(1, 6) : it % 2 ? draw(1, 90) : 16 * draw(1, 10), 0, 0, 0};
            if (i < nm + nn) order[2].push_back(i);
            if (i < nm || i >= nm + nn) order[0].push_back(i);
            if (i >= nm) order[1].push_back(i);
        }
        int64_t elems[3];
        for (int t = 0; t < 3; ++t) {
            std::shuffle(order[t].begin(), order[t].end(), r);
            int64_t at = 1;
            for (int x : order[t]) {
                (t == 0 ? L[x].sa : t == 1 ? L[x].sb : L[x].sc) = at;
                at *= L[x].size;
            }
            elems[t] = at;
        }
        for (int dtype : {TTX_F32, TTX_F64})
            for (int v = 0; v < kContractVariants; ++v) {
                ContractPlan p;
                plan_contraction_as(dtype, L.data(), c, v, draw(1, 3), false, &p);
                const int es = dtype == TTX_F32 ? 4 : 8;
                const int64_t bx = elems[p.swapped ? 1 : 0] * es, by = elems[p.swapped ? 0 : 1] * es;
                vec += p.vec_xy;
                wide += v == 3 && p.vec_xy && !p.yk;
                if (dtype == TTX_F32 ? in_bounds<float>(p, bx, by) : in_bounds<double>(p, bx, by)) continue;
                std::printf("FAIL: read out of range; %d-byte elements, tile shape %d\n", es, v);
                for (const auto& l : L)
                    std::printf("  extent %lld, strides %lld, %lld and %lld\n", (long long)l.size, (long long)l.sa,
                                (long long)l.sb, (long long)l.sc);
                return 1;
            }
    }
    std::printf("ok: %d contractions, %d whole-unit plans, %d with 80 columns along their run, "
                "%lld lanes in the walk and %lld beyond\n",
                count, vec, wide, (long long)replayed[0], (long long)replayed[1]);
    return 0;
}
