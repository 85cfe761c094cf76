// Planning of a direct contraction (host only): which operand gives the
// product's rows, the digit orders of the three label groups, the tile shape
// and the splits of the contracted index.
#include <algorithm>
#include <vector>

#include "contract.h"
#include "ttx_internal.h"

namespace ttx {
namespace {

struct Lab {
    int64_t size, s0, s1;   // extent, strides in the group's first and second tensor
};

constexpr int kCUs = 256;
// 64 lanes' addresses leave a CU's address unit as 64-byte segments, about one a cycle.
constexpr double kSegmentBytes = 64.0;
constexpr double kDramBytesPerCycle = 2300.0;   // 5.5 TB/s at 2.4 GHz
constexpr double kStepCycles = 1500.0;          // latency of one k step (loads from L2, a barrier)
constexpr double kTileCycles = 9000.0;          // start and end of a tile: tables, first loads, stores of C
constexpr double kLaunchCycles = 10000.0;       // a second launch

// Fuses neighbours that are contiguous in both tensors (Sec. 2.1's merging).
void merge(std::vector<Lab>& g) {
    for (size_t i = 0; i + 1 < g.size();) {
        if (g[i + 1].s0 == g[i].s0 * g[i].size && g[i + 1].s1 == g[i].s1 * g[i].size) {
            g[i].size *= g[i + 1].size;
            g.erase(g.begin() + i + 1);
        } else {
            ++i;
        }
    }
}

int find_unit(const std::vector<Lab>& g, bool second) {   // the label with stride 1, -1 if none
    for (size_t i = 0; i < g.size(); ++i)
        if ((second ? g[i].s1 : g[i].s0) == 1) return int(i);
    return -1;
}

// Two demands on a CU that overlap, but not perfectly.
double overlap(double a, double b) { return std::max(a, b) + 0.3 * std::min(a, b); }

double waste(int64_t size, int64_t chunk) { return double((size + chunk - 1) / chunk * chunk) / double(size); }

void put(ContractGroup* g, int64_t size, int64_t s0, int64_t s1, int guard, int64_t weight) {
    if (size <= 1 && guard < 0) return;
    ContractDigit& d = g->d[g->nd++];
    d.size = size;
    d.dv.init(size < (int64_t(1) << 32) ? uint32_t(size) : 1u);
    d.s0 = s0;
    d.s1 = s1;
    d.guard = guard;
    d.weight = weight;
    g->total *= size;
}

// The group's digits: the chunks of up to two labels first (cut[i]: label,
// chunk), then every label in order with the rest of the cut ones in their place.
struct Cut {
    int label;
    int64_t chunk;
};
void fill(ContractGroup* g, const std::vector<Lab>& labs, const std::vector<Cut>& cuts) {
    *g = ContractGroup();
    g->total = 1;
    g->guard_ext[0] = g->guard_ext[1] = int64_t(1) << 62;
    for (size_t c = 0; c < cuts.size(); ++c) {
        const Lab& l = labs[cuts[c].label];
        g->guard_ext[c] = l.size;
        put(g, cuts[c].chunk, l.s0, l.s1, int(c), 1);
    }
    for (size_t i = 0; i < labs.size(); ++i) {
        int guard = -1;
        int64_t chunk = 1;
        for (size_t c = 0; c < cuts.size(); ++c)
            if (cuts[c].label == int(i)) guard = int(c), chunk = cuts[c].chunk;
        const int64_t rest = (labs[i].size + chunk - 1) / chunk;
        if (guard >= 0 && rest == 1) continue;   // the chunk is the whole label
        put(g, rest, labs[i].s0 * chunk, labs[i].s1 * chunk, guard, chunk);
    }
    g->wide = g->total >= (int64_t(1) << 32);
}

struct Groups {
    std::vector<Lab> m, n, k;
    bool swapped = false;
    int y = -1, x = -1;     // rows: C's and X's stride-1 labels (x == y where they are one)
    int w = -1;             // columns: Y's stride-1 label
    int kx = -1, ky = -1;   // contracted: X's and Y's stride-1 labels
    double sm = 1, sn = 1, sk = 1;
};

Groups group_labels(const ContractLabel* labels, int count) {
    Groups g;
    bool lead_in_b = false;
    for (int i = 0; i < count; ++i)
        if (labels[i].size > 1 && labels[i].sc == 1 && labels[i].sb != 0) lead_in_b = true;
    g.swapped = lead_in_b;
    for (int i = 0; i < count; ++i) {
        const ContractLabel& l = labels[i];
        if (l.size <= 1) continue;
        const int64_t sx = lead_in_b ? l.sb : l.sa, sy = lead_in_b ? l.sa : l.sb;
        if (l.sc == 0) g.k.push_back(Lab{l.size, sx, sy});
        else if (sx != 0) g.m.push_back(Lab{l.size, sx, l.sc});
        else g.n.push_back(Lab{l.size, sy, l.sc});
    }
    auto by1 = [](const Lab& a, const Lab& b) { return a.s1 < b.s1; };
    auto by0 = [](const Lab& a, const Lab& b) { return a.s0 < b.s0; };
    std::sort(g.m.begin(), g.m.end(), by1);
    std::sort(g.n.begin(), g.n.end(), by1);
    std::sort(g.k.begin(), g.k.end(), by0);
    merge(g.m);
    merge(g.n);
    merge(g.k);
    g.y = find_unit(g.m, true);
    g.x = find_unit(g.m, false);
    g.w = find_unit(g.n, false);
    g.kx = find_unit(g.k, false);
    g.ky = find_unit(g.k, true);
    for (const Lab& l : g.m) g.sm *= double(l.size);
    for (const Lab& l : g.n) g.sn *= double(l.size);
    for (const Lab& l : g.k) g.sk *= double(l.size);
    return g;
}

// Whether every `unit` places of the walk that starts with the group's digits
// (the cut label's chunk, where there is one) are one run of a tensor: the
// run's length and, where it is cut, the label's extent are whole units.
bool whole_units(int64_t run, int64_t extent, int unit) { return run % unit == 0 && extent % unit == 0; }

// Segments that a run of `run` elements of `es` bytes costs per element.
double per_element(double run, int es) { return 1.0 / std::min(std::max(run, 1.0), kSegmentBytes / es); }

// Rows, columns and contracted digits for one tile shape; returns the cycles
// one full tile keeps a CU busy.  packed: the operands are read as packed
// tiles, so only C's order counts.
double shape(const Groups& g, int es, int mb, int nb, bool packed, ContractPlan* p) {
    const int MT = 64 * mb, NT = 16 * nb, KT = contract_kt(es, mb), U = 16 / es;
    ContractArgs& a = p->args;
    a.rows = MT;
    a.walk_x = a.walk_y = a.kwalk_x = a.kwalk_y = a.c_cut = 1;
    p->packed = packed;
    p->xk = g.kx >= 0 && g.x < 0;
    p->yk = g.ky >= 0 && g.w < 0;
    bool vec_x = false, vec_y = false, vec_c = false;
    double run_x = 1, run_y = 1;   // elements in a row of X's and Y's loads

    // contracted: X's run first, or Y's; where both run along k over different
    // labels, a few of each
    std::vector<Lab> k = g.k;
    if (p->xk && p->yk && g.kx != g.ky) {
        auto chunk = [](int64_t s, int64_t most) {
            for (int64_t c = most; c > 1; c /= 2)
                if (c <= s && waste(s, c) <= 1.13) return c;
            return int64_t(1);
        };
        const int64_t cx = chunk(k[g.kx].size, 4), cy = chunk(k[g.ky].size, KT / 4 < 4 ? KT / 4 : 4);
        fill(&a.k, k, {Cut{g.kx, cx}, Cut{g.ky, cy}});
        a.kwalk_x = int(cx);
        a.kwalk_y = int(cy);
        run_x = double(cx);
        run_y = double(cy);
        vec_x = whole_units(cx, k[g.kx].size, U);
        vec_y = whole_units(cy, k[g.ky].size, U);
    } else {
        const int lead = p->xk ? g.kx : p->yk ? g.ky : -1;
        if (lead > 0) std::rotate(k.begin(), k.begin() + lead, k.begin() + lead + 1);
        fill(&a.k, k, {});
        const double run = lead >= 0 ? std::min(double(k[0].size), double(KT)) : 1.0;
        const bool whole = lead >= 0 && whole_units(k[0].size, k[0].size, U);
        if (p->xk) run_x = run, vec_x = whole;
        if (p->yk) run_y = run, vec_y = whole;
    }
    const double K = double(a.k.total);

    // columns: in C's order but for a chunk of Y's run (a power of two: it
    // divides the tile's columns), which comes first
    if (g.w <= 0 || packed) {
        fill(&a.n, g.n, {});
        if (g.w == 0) {
            run_y = std::min(double(g.n[0].size), double(NT));
            vec_y = whole_units(g.n[0].size, g.n[0].size, U);
        }
    } else {
        const int64_t want = K >= 64 ? 16 : 4;
        for (int64_t c = 2; c <= std::min(want, g.n[g.w].size); c *= 2)
            if (waste(g.n[g.w].size, c) <= 1.07) a.c_cut = int(c);
        fill(&a.n, g.n, {Cut{g.w, a.c_cut}});
        run_y = double(a.c_cut);
        vec_y = whole_units(a.c_cut, g.n[g.w].size, U);
    }

    // rows: C's run and, where X runs along another row label, a chunk of each.
    // Where the rows hold whole runs of C and the columns go on where they end,
    // a kernel that walks C in its own order has runs of both.
    const bool one_step = contract_has_short(es, mb, nb) && a.k.total <= KT;
    const double cs = 2.0;   // accesses per element of C
    const double seg = one_step ? 3.0 : 1.0;
    const double flops = K * MT * NT * 2 / (es == 4 ? 256.0 : 128.0);
    auto adjacent = [&](int64_t run) { return one_step && run <= MT && !g.n.empty() && g.n[0].s1 == run; };
    auto c_run = [&](int64_t run) { return adjacent(run) ? double(run) * NT / a.c_cut : double(run); };
    auto cost = [&](double rows, double rx, double rc) {
        const double loads = packed ? (rows + NT) * K / (64.0 / es)
                                    : rows * K * per_element(rx, es) + NT * K * per_element(run_y, es);
        return overlap(flops, seg * loads + cs * rows * NT * per_element(rc, es));
    };
    int run = 0;   // rows of C's walk before it turns to the columns (0: all)
    double cycles;
    if (!packed && g.x >= 0 && g.y >= 0 && g.x != g.y) {
        const int64_t ex = g.m[g.x].size, ey = g.m[g.y].size;
        double best = 1e300;
        int64_t bx = 1, by = 1;
        for (int64_t cx = 1; cx <= std::min<int64_t>(32, ex); ++cx)
            for (int64_t cy = 1; cy <= std::min<int64_t>(64, ey) && cx * cy <= MT; ++cy) {
                const double used = double(cx * cy * (MT / (cx * cy)));
                const double extra = waste(ex, cx) * waste(ey, cy) * MT / used;
                const double odd = (whole_units(cx, ex, U) ? 1.0 : 1.1) * (whole_units(cy, ey, 4) ? 1.0 : 1.2);
                const double rc = cy == ey ? c_run(ey) : double(cy);
                const double c = extra * odd * (cost(used, double(cx), rc) + kTileCycles / 4);
                if (c < best) best = c, bx = cx, by = cy;
            }
        fill(&a.m, g.m, {Cut{g.y, by}, Cut{g.x, bx}});
        a.walk_x = int(bx);
        a.walk_y = int(by);
        a.rows = int(bx * by * (MT / (bx * by)));
        vec_x = whole_units(bx, ex, U);
        vec_c = whole_units(by, ey, 4);
        if (by == ey && adjacent(ey)) run = int(ey);
        cycles = cost(a.rows, double(bx), by == ey ? c_run(ey) : double(by));
    } else {
        fill(&a.m, g.m, {});
        int64_t lead = 1;   // rows that are one run of C
        for (const Lab& l : g.m)
            if (l.s1 == lead) lead *= l.size;
        if (g.x >= 0) {
            run_x = g.x == 0 ? std::min(double(g.m[0].size), double(MT)) : 1.0;
            vec_x = g.x == 0 && whole_units(g.m[0].size, g.m[0].size, U);
        }
        vec_c = whole_units(lead, lead, 4);
        if (adjacent(lead)) {
            run = int(lead);
            a.rows = int(lead * (MT / lead));
        }
        cycles = cost(a.rows, run_x, std::min(c_run(lead), double(MT)));
    }
    a.dv_run.init(uint32_t(run ? run : a.rows));
    a.dv_cut.init(uint32_t(NT / a.c_cut));
    p->vec_xy = vec_x && vec_y;
    p->vec_c = vec_c;
    a.tiles_m = (a.m.total + a.rows - 1) / a.rows;
    a.tiles_n = (a.n.total + NT - 1) / NT;
    a.steps = g.sk == 0 ? 0 : (a.k.total + KT - 1) / KT;
    return cycles;
}

void set_splits(ContractPlan* p, int splits) {
    ContractArgs& a = p->args;
    a.split_steps = a.steps ? (a.steps + splits - 1) / splits : 0;
    p->splits = a.split_steps ? int((a.steps + a.split_steps - 1) / a.split_steps) : 1;
    const int64_t tiles = a.tiles_m * a.tiles_n;
    a.dv_m.init(uint32_t(std::min<int64_t>(a.tiles_m, 0xffffffff)));
    a.dv_tiles.init(uint32_t(std::min<int64_t>(tiles, 0xffffffff)));
}

const ContractVariant kMenu[] = {
#define TTX_V(i, mb, nb) {mb, nb},
    TTX_CONTRACT_MENU(TTX_V)
#undef TTX_V
};

void start(int dtype, const ContractLabel* labels, int count, Groups* g, ContractPlan* p) {
    *g = group_labels(labels, count);
    for (int i = 0; i < count; ++i)
        if (labels[i].size == 0 && labels[i].sc == 0) g->sk = 0;   // an empty sum
    p->dtype = dtype;
    p->swapped = g->swapped;
}

}  // namespace

void plan_contraction_as(int dtype, const ContractLabel* labels, int count, int variant, int splits, bool packed,
                         ContractPlan* out) {
    Groups g;
    start(dtype, labels, count, &g, out);
    out->variant = variant;
    shape(g, elem_bytes(dtype), kMenu[variant].mb, kMenu[variant].nb, packed, out);
    set_splits(out, splits);
}

// The tile shape, splits and packing with the least estimated time: matrix or
// address cycles of the CU with the most tiles (a last wave that fills a few
// CUs costs as much as a full one, which is what 80 columns are for), or the
// latency of the k steps where few workgroups run (128 x 96 results, k = 2048:
// 16 us in 16 splits, 69 in one), or C's traffic.  80 columns were taken for 46
// of 153 FP32 products and contractions of long sums; without that shape those
// take 1.06 times as long (0.81 to 1.58; m = n = k = 1600: 88 us against 79).
// In FP64 the 48 that take it would do as well without (0.997; 0.86 to 1.34).  Packing the operands of a short sum costs a launch and pays where
// many tiles read them in short runs (24^6 FP32 results, sums of 16: 309 us
// against 326; with beta = 0 150 against 212).  Over 25 shapes in both types
// the choice was within 10% of the best of the menu on 22.
void plan_contraction(int dtype, const ContractLabel* labels, int count, int64_t ws_elems, ContractPlan* out) {
    Groups g;
    const int es = elem_bytes(dtype);
    double best = 1e300;
    int best_v = 0, best_s = 1;
    bool best_p = false;
    for (int v = 0; v < kContractVariants; ++v)
        for (bool packed : {false, true}) {
            ContractPlan p;
            start(dtype, labels, count, &g, &p);
            const int mb = kMenu[v].mb, nb = kMenu[v].nb, KT = contract_kt(es, mb);
            const bool one_step = contract_has_short(es, mb, nb) && g.sk > 0 && g.sk <= KT;
            if (packed && !one_step) continue;
            const double cycles = shape(g, es, mb, nb, packed, &p);
            const double tiles = double(p.args.tiles_m) * double(p.args.tiles_n);
            const double area = 64.0 * mb * 16.0 * nb, out_bytes = g.sm * g.sn * es;
            const double panels = (double(p.args.tiles_m) * 64.0 * mb + double(p.args.tiles_n) * 16.0 * nb) * KT;
            if (packed && panels > double(ws_elems)) continue;
            const int per_cu = one_step || mb * nb < 4 ? 4 : 3;
            for (int s = 1; s <= 64; s = s < 8 ? s + 1 : s * 2) {
                if (s > 1 && (p.args.steps < 2 * s || double(s) * tiles * area > double(ws_elems))) break;
                const double steps = double((p.args.steps + s - 1) / s);
                const double frac = p.args.steps ? steps / double(p.args.steps) : 1.0;
                const double wgs = tiles * s;
                // a tile's latency is hidden behind the others on its CU, more
                // so where C is asked for first
                const double whole = one_step ? kTileCycles / 2 : kTileCycles, own = whole / per_cu;
                const double busy = double(int64_t((wgs + kCUs - 1) / kCUs)) * (cycles * frac + own);
                const double wait = double(int64_t((wgs + kCUs * per_cu - 1) / (kCUs * per_cu))) *
                                    (steps * kStepCycles + whole);
                double c = overlap(std::max(busy, wait), 2.0 * out_bytes / kDramBytesPerCycle);
                if (s > 1) c += kLaunchCycles + 500.0 * s + (2.0 * s * tiles * area * es + 2.0 * out_bytes) / kDramBytesPerCycle;
                if (packed) c += kLaunchCycles + 2.0 * panels * es / kDramBytesPerCycle;
                // a sum of one step with a shape that has no kernel for it: C is
                // asked for last and in pieces of lines (16^6 FP64 results, sums
                // of 8: 58 us against 45)
                if (p.args.steps == 1 && !one_step) c *= 1.25;
                if (c < best) best = c, best_v = v, best_s = s, best_p = packed;
            }
        }
    plan_contraction_as(dtype, labels, count, best_v, best_s, best_p, out);
}

hipError_t launch_contraction(const ContractPlan& p, const void* A, const void* B, void* C, void* workspace,
                              double alpha, double beta, hipStream_t stream) {
    const void* X = p.swapped ? B : A;
    const void* Y = p.swapped ? A : B;
    if (p.dtype == TTX_F32)
        return launch_contract_f32(p, static_cast<const float*>(X), static_cast<const float*>(Y),
                                   static_cast<float*>(C), static_cast<float*>(workspace), float(alpha), float(beta),
                                   stream);
    return launch_contract_f64(p, static_cast<const double*>(X), static_cast<const double*>(Y),
                               static_cast<double*>(C), static_cast<double*>(workspace), alpha, beta, stream);
}

}  // namespace ttx
