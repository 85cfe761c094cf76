// The box tiles of large problems (some 10^5 to 10^6 elements, up to 4 units a
// thread) on the CPU; see box_sim.cpp.  box_sim_large SEED COUNT
#define main box_sim_main
#include "box_sim.cpp"
#undef main

int main(int argc, char** argv) {
    std::mt19937 r(argc > 1 ? std::atoi(argv[1]) : 0);
    const int count = argc > 2 ? std::atoi(argv[2]) : 10;
    auto draw = [&](int lo, int hi) { return int(r() % uint32_t(hi - lo + 1)) + lo; };
    int done[8] = {}, cut = 0;   // by type; with an index that is cut and leaves a remainder
    for (int it = 0, drawn = 0; it < count; ++drawn) {
        if (drawn >= 100 * count) return 1;
        const int n = draw(2, 4), code = it % 8;
        std::vector<int> perm(n);
        std::iota(perm.begin(), perm.end(), 0);
        std::shuffle(perm.begin(), perm.end(), r);
        std::vector<int64_t> size(n), oa(n), ob(n);
        const int most = n == 2 ? 1000 : n == 3 ? 100 : 32;
        for (int d = 0; d < n; ++d) size[d] = draw(most / 2, most);
        const bool leading = draw(0, 3) == 0;
        for (int d = 0; d < n; ++d) oa[d] = size[d] + (leading ? draw(0, 3) : 0);
        for (int k = 0; k < n; ++k) ob[k] = size[perm[k]] + (leading ? draw(0, 3) : 0);
        Problem p;
        BoxPlan bp;
        if (make_problem(code, n, perm.data(), size.data(), oa.data(), ob.data(), &p) != TTX_OK) continue;
        if (!plan_box(p, drawn & 1, &bp) || bp.units != 4) continue;
        ++it;
        ++done[code];
        cut += bp.s.sizeA % bp.s.tA || bp.s.sizeB % bp.s.tB;
        const int ua = 16 / elem_bytes(p.dtype_a), ub = 16 / elem_bytes(p.dtype);
        if (ua == 4) ub == 4 ? simulate<4, 4>(p, bp) : simulate<4, 2>(p, bp);
        else if (ua == 2) ub == 4 ? simulate<2, 4>(p, bp) : ub == 2 ? simulate<2, 2>(p, bp) : simulate<2, 1>(p, bp);
        else ub == 2 ? simulate<1, 2>(p, bp) : simulate<1, 1>(p, bp);
    }
    std::printf("ok: four units a thread, by type");
    for (int n : done) std::printf(" %d", n);
    std::printf(", %d with remainders\n", cut);
    return 0;
}
