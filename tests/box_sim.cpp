// Runs the box tiles of random problems on the CPU: every unit of every
// thread, with the planner and the offsets that the kernel uses, against the
// transposition's definition.  box_sim SEED COUNT
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <numeric>
#include <random>
#include <string>
#include <vector>

#include "box.h"
#include "ttx_internal.h"

using namespace ttx;

namespace ttx {
ttx_status fail(ttx_status s, const std::string&) { return s; }
}  // namespace ttx

static void stop(const char* what, const Problem& p) {
    std::printf("FAIL: %s; code %d\n", what, p.code);
    for (int d = 0; d < p.n; ++d)
        std::printf("  extent %lld, strides %lld and %lld\n", (long long)p.dim[d].size, (long long)p.dim[d].sa,
                    (long long)p.dim[d].sb);
    std::exit(1);
}

template <int UA, int UB>
static void simulate(const Problem& p, const BoxPlan& bp) {
    const BoxShape& s = bp.s;
    const int64_t na = p.extent_a / elem_bytes(p.dtype_a), nb = p.extent_b / elem_bytes(p.dtype);
    std::vector<int64_t> want(nb, -1), got(nb, -1), c(p.n, 0), lds(box_lds(elem_bytes(p.dtype), bp.units));
    for (int64_t e = 0; e < p.elements; ++e) {
        int64_t oa = 0, ob = 0;
        for (int d = 0; d < p.n; ++d) oa += c[d] * p.dim[d].sa, ob += c[d] * p.dim[d].sb;
        want[ob] = oa;
        for (int d = 0; d < p.n && ++c[d] == p.dim[d].size; ++d) c[d] = 0;
    }
    auto at = [&](int l) {   // the LDS element, in bounds
        l += l >> s.skew;
        if (l < 0 || l >= int(lds.size())) stop("LDS bounds", p);
        return l;
    };
    std::vector<BoxUnits<UA, UB>> u(kThreads);
    std::vector<int32_t> by(nb, -1);
    for (uint32_t t = 0; t < s.ntiles; ++t) {
        const BoxCoord b = box_coord(s, t);
        for (int tid = 0; tid < kThreads; ++tid) u[tid].init(s, tid, b);
        auto write = [&](int64_t ob, int64_t value) {
            if (ob < 0 || ob >= nb || want[ob] != value) stop("value", p);
            if (by[ob] >= 0 && by[ob] != int32_t(t)) stop("written by two boxes", p);
            got[ob] = value;
            by[ob] = int32_t(t);
        };
        if (u[0].shorter) {
            int n = 1;
            for (int k = 0; k < s.nB; ++k) n *= BoxUnits<1, 1>::extent(s.dB[k], b);
            for (int e = 0; e < n; ++e) {
                int64_t oa = b.oa, ob = b.ob;
                for (int k = 0, v = e; k < s.nB; ++k) {
                    const int ext = BoxUnits<1, 1>::extent(s.dB[k], b);
                    oa += int64_t(v % ext) * s.dB[k].sa;
                    ob += int64_t(v % ext) * s.dB[k].sb;
                    v /= ext;
                }
                write(ob, oa);
            }
            continue;
        }
        std::fill(lds.begin(), lds.end(), -1);
        if (u[0].nua > bp.units * kThreads || u[0].nub > bp.units * kThreads) stop("units", p);
        for (int i = 0; i < bp.units; ++i)
            for (int tid = 0; tid < kThreads && kThreads * i < u[0].nua; ++tid)
                for (int j = 0; j < UA; ++j) {
                    const int64_t a = int64_t(b.oa) + u[tid].rel_a[i] + j;
                    if (a < 0 || a >= na) stop("A bounds", p);
                    if (u[tid].whole_a && (s.skew != 31 || u[tid].lds_a[i] % UA)) stop("LDS alignment", p);
                    int64_t& x = lds[at(u[tid].put(i, j))];
                    if (x >= 0 && x != a) stop("LDS clash", p);
                    x = a;
                }
        for (int i = 0; i < bp.units; ++i)
            for (int tid = 0; tid < kThreads && kThreads * i < u[0].nub; ++tid)
                for (int j = 0; j < UB; ++j) {
                    const int l = u[tid].gather(i, j);
                    if (l < 0 || l >= int(lds.size())) stop("LDS bounds", p);
                    write(int64_t(b.ob) + u[tid].rel_b[i] + j, lds[l]);
                }
    }
    if (got != want) stop("coverage", p);
}

int main(int argc, char** argv) {
    std::mt19937 r(argc > 1 ? std::atoi(argv[1]) : 0);
    const int count = argc > 2 ? std::atoi(argv[2]) : 100;
    auto draw = [&](int lo, int hi) { return int(r() % uint32_t(hi - lo + 1)) + lo; };
    int done = 0, filled = 0, skewed = 0, small = 0;
    for (int it = 0; it < count; ++it) {
        const int n = draw(2, 6);
        std::vector<int> perm(n);
        std::iota(perm.begin(), perm.end(), 0);
        if (draw(0, 9)) std::shuffle(perm.begin(), perm.end(), r);   // else flat, or rows with a distance
        std::vector<int64_t> size(n), oa(n), ob(n);
        int64_t total = 1;
        for (int d = 0; d < n; ++d) {
            size[d] = draw(1, int(std::min<int64_t>(draw(0, 2) ? 40 : 700, std::max<int64_t>(1, 60000 / total))));
            total *= size[d];
        }
        std::shuffle(size.begin(), size.end(), r);
        const bool leading = total < 8000 && draw(0, 2) == 0;
        for (int d = 0; d < n; ++d) oa[d] = size[d] + (leading ? draw(0, 3) : 0);
        for (int k = 0; k < n; ++k) ob[k] = size[perm[k]] + (leading ? draw(0, 3) : 0);
        Problem p;
        BoxPlan bp;
        if (make_problem(draw(0, 7), n, perm.data(), size.data(), oa.data(), ob.data(), &p) != TTX_OK) continue;
        if (!plan_box(p, it & 1, &bp, it % 3 == 0)) continue;   // a third as in a launch over many problems
        if (it % 3 == 0 && bp.units != 2) stop("more than two units a thread", p);
        ++done;
        filled += bp.s.tC > 1;
        skewed += bp.s.skew < 31;
        small += bp.units == 2;
        const int ua = 16 / elem_bytes(p.dtype_a), ub = 16 / elem_bytes(p.dtype);
        if (ua == 4) ub == 4 ? simulate<4, 4>(p, bp) : simulate<4, 2>(p, bp);
        else if (ua == 2) ub == 4 ? simulate<2, 4>(p, bp) : ub == 2 ? simulate<2, 2>(p, bp) : simulate<2, 1>(p, bp);
        else ub == 2 ? simulate<1, 2>(p, bp) : simulate<1, 1>(p, bp);
    }
    std::printf("ok: %d boxes of %d problems, %d filled, %d skewed, %d small\n", done, count, filled, skewed, small);
    return 0;
}
