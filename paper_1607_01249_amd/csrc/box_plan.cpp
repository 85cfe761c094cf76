// Choice of a box tile (host only; see box.h).  Every pair of candidate runs
// gives a box, small ones also filled up by a third index; the cheapest by an
// estimate of its time is taken (4 to 6 us of host time, up to 30).
#include <algorithm>
#include <cmath>
#include <cstring>

#include "box.h"
#include "ttx_internal.h"

namespace ttx {
namespace {

constexpr int kBoxBytes = 16384;

// a / b and its ceiling for the sizes here (extents of tensors below 4 GiB):
// divisions of 64 bits took a third of a choice's time.
int64_t quotient(int64_t a, int64_t b) { return uint32_t(a) / uint32_t(b); }
int64_t ceiling(int64_t a, int64_t b) { return quotient(a + b - 1, b); }

// One side's run: its first `whole` indices and `t` steps of the next one.
struct Run {
    int whole;
    int64_t t;       // 1 .. extent - 1, or 0: no split index
    int64_t len;
};

// Candidate runs of about 64 bytes to 4 KiB along `order` (A's or B's): their
// whole indices, and pieces of the next one (whole 128-byte lines of a long
// stride-1 index, else near-even pieces).  A run that can't go on because the
// next index doesn't follow in memory may be shorter.
int runs_of(const Problem& p, const int* order, bool in_a, int es, Run* out, int cap) {
    int n = 0;
    int64_t len = 1;
    const int64_t most = kBoxBytes / es, line = 128 / es;
    auto follows = [&](int k) {
        if (k >= p.n) return false;
        const Dim &d = p.dim[order[k]], &e = p.dim[order[k - 1]];
        return in_a ? d.sa == e.sa * e.size : d.sb == e.sb * e.size;
    };
    for (int k = 0; n < cap && (k == 0 || follows(k)); ++k) {
        const Dim& d = p.dim[order[k]];
        int64_t last = 0;
        for (int64_t want = 64; want <= 4096 && n < cap; want *= 2) {
            int64_t t = std::max<int64_t>(1, quotient(quotient(want, es), len));
            if (t >= d.size || len * t > most) break;
            if (len != 1 || t & (line - 1) || d.size < 4 * t) t = ceiling(d.size, ceiling(d.size, t));
            if (t == last || t >= d.size) continue;
            last = t;
            out[n++] = Run{k, t, len * t};
        }
        if (len * d.size > most) break;
        len *= d.size;
        if ((len * es >= 64 || !follows(k + 1)) && n < cap) out[n++] = Run{k + 1, 0, len};
        if (len * es >= 4096) break;
    }
    return n;
}

// One box: its extents t (by index), the runs they give and what they cost.
struct Box {
    int t[kMaxDims];
    int volume, LA, LB;          // elements of the box and of its runs
    int sa, sb, sc;              // indices that the runs cut, and a third one that the box cuts, -1: none
    int in_run_a, in_run_b;      // positions (A's order, B's order) that a run holds
    int nua, nub;                // units of a full box
    double tiles;
};

// Boxes along index d; most indices need no division.
int64_t steps_of(const Problem& p, const Box& b, int d) {
    const int64_t size = p.dim[d].size, t = b.t[d];
    return t == 1 ? size : t == size ? 1 : ceiling(size, t);
}

// Fills in a box from its extents; false where the kernel can't take it.
bool box_of(const Problem& p, Box* b) {
    const int ea = elem_bytes(p.dtype_a), eb = elem_bytes(p.dtype);
    const int UA = 16 / ea, UB = 16 / eb;
    const int* t = b->t;
    int dims = 0;
    b->volume = 1;
    for (int d = 0; d < p.n; ++d) {
        b->volume *= t[d];
        dims += t[d] > 1;
    }
    if (dims > kBoxDims || b->volume * eb > kBoxBytes || b->volume * ea > 2 * kBoxBytes) return false;
    // a run: whole indices that follow each other in memory, and part of the next
    b->LA = b->LB = 1;
    b->sa = b->sb = -1;
    b->in_run_a = b->in_run_b = 0;
    for (int k = 0; k < p.n; ++k) {
        if (k > 0 && p.dim[k].sa != p.dim[k - 1].sa * p.dim[k - 1].size) break;
        b->LA *= t[k];
        b->in_run_a = k + 1;
        if (t[k] < p.dim[k].size) {
            b->sa = k;
            break;
        }
    }
    for (int k = 0; k < p.n; ++k) {
        const int d = p.perm[k];
        if (k > 0 && p.dim[d].sb != p.dim[p.perm[k - 1]].sb * p.dim[p.perm[k - 1]].size) break;
        b->LB *= t[d];
        b->in_run_b = k + 1;
        if (t[d] < p.dim[d].size) {
            b->sb = d;
            break;
        }
    }
    if (b->LA < UA || b->LB < UB) return false;
    // of the indices outside the runs one may be cut
    b->sc = -1;
    for (int d = 0; d < p.n; ++d)
        if (t[d] > 1 && t[d] < p.dim[d].size && d != b->sa && d != b->sb) {
            if (b->sc >= 0) return false;
            b->sc = d;
        }
    const int runs_a = b->volume / b->LA, runs_b = b->volume / b->LB;
    b->nua = runs_a * ((b->LA + UA - 1) / UA);
    b->nub = runs_b * ((b->LB + UB - 1) / UB);
    if (b->nua > kThreads * kBoxUnits || b->nub > kThreads * kBoxUnits) return false;
    if (runs_a * (b->LA + 1) + UA > box_lds(eb, kBoxUnits)) return false;   // with an odd pitch
    b->tiles = 1;
    for (int d = 0; d < p.n; ++d) b->tiles *= double(steps_of(p, *b, d));
    return true;
}

// Whether two units per thread hold the box.
bool small_box(const Problem& p, const Box& b) {
    const int UA = 16 / elem_bytes(p.dtype_a);
    return b.nua <= 2 * kThreads && b.nub <= 2 * kThreads &&
           b.volume / b.LA * (b.LA + 1) + UA <= box_lds(elem_bytes(p.dtype), 2);
}

// Whether every run of B is whole 128-byte lines (for a B that starts on one).
bool whole_lines_b(const Problem& p, const Box& b) {
    const int eb = elem_bytes(p.dtype);
    bool lines = b.LB * eb % 128 == 0;
    for (int k = b.in_run_b; k < p.n; ++k) lines = lines && p.dim[p.perm[k]].sb * eb % 128 == 0;
    return lines;
}

// Estimated time in microseconds: the bytes at the rate of a large copy; per
// run up to half a 128-byte line (less where runs are whole lines, or where the
// next boxes in B's order go on with them, so that the shared line is still in
// the L2); a byte or so per unit (addresses, LDS) and a fixed cost per box; and
// what one compute unit's boxes wait for, which counts where there are few.
// The constants are fitted to the times of some 9000 boxes of 190 problems on
// buffers that the caches don't hold; the boxes taken come to 3.27 ms where the
// best of all come to 3.16 ms.
double box_cost(const Problem& p, bool beta0, const Box& b) {
    const int ea = elem_bytes(p.dtype_a), eb = elem_bytes(p.dtype);
    const double n = double(p.elements), sides = beta0 ? 1.0 : 2.0;   // accesses of B
    // boxes between one box and the one that goes on with its run of A or B
    double da = 1.0, db = 1.0;
    for (int k = 0, d; b.sa >= 0 && (d = p.perm[k]) != b.sa; ++k) da *= double(steps_of(p, b, d));
    for (int k = 0, d; b.sb >= 0 && (d = p.perm[k]) != b.sb; ++k) db *= double(steps_of(p, b, d));
    bool lines_a = b.LA * ea % 128 == 0;
    const bool lines_b = whole_lines_b(p, b);
    for (int k = b.in_run_a; k < p.n; ++k) lines_a = lines_a && p.dim[k].sa * ea % 128 == 0;
    const double runs_a = n / double(b.LA) * (lines_a ? 36.0 : b.sa >= 0 && da <= 8.0 ? 21.0 : 57.0);
    const double runs_b = n / double(b.LB) * (lines_b ? 4.0 : b.sb >= 0 && db <= 8.0 ? 27.0 : 49.0) * sides;
    const double units = 0.8 * double(b.nua + b.nub) * b.tiles;
    const double wide = small_box(p, b) ? 1.0 : beta0 ? 1.084 : 1.076;
    const double bytes = (n * (ea + eb * sides) + runs_a + runs_b + units) * wide + 1200.0 * b.tiles;
    const double rounds = std::ceil(b.tiles / 256.0), fill = std::ceil(double(std::max(b.nua, b.nub)) / kThreads);
    return bytes / 6e6 + 0.026 * fill * (1.0 + 0.02 * (rounds - 1.0));
}

template <typename F>
void each_box(const Problem& p, F&& f) {
    const int ea = elem_bytes(p.dtype_a), eb = elem_bytes(p.dtype);
    int id[kMaxDims];
    for (int d = 0; d < p.n; ++d) id[d] = d;
    Run ra[24], rb[24];
    const int na = runs_of(p, id, true, ea, ra, 24), nb = runs_of(p, p.perm, false, eb, rb, 24);
    for (int i = 0; i < na; ++i)
        for (int j = 0; j < nb; ++j) {
            Box b;
            for (int d = 0; d < p.n; ++d) b.t[d] = 1;
            for (int k = 0; k < ra[i].whole; ++k) b.t[k] = int(p.dim[k].size);
            if (ra[i].t) b.t[ra[i].whole] = int(ra[i].t);
            for (int k = 0; k < rb[j].whole; ++k) b.t[p.perm[k]] = int(p.dim[p.perm[k]].size);
            if (rb[j].t) b.t[p.perm[rb[j].whole]] = std::max(b.t[p.perm[rb[j].whole]], int(rb[j].t));
            if (!box_of(p, &b)) continue;
            f(b);
            // a small box filled up to two, then four units a thread, with the
            // next indices of A's order or of B's: whole ones, then part of one
            for (int side = 0; side < 2 && std::max(b.nua, b.nub) <= kThreads; ++side) {
                Box c = b, e;
                int k = 0;
                for (int most = 2 * kThreads; most <= 4 * kThreads && k < p.n; most *= 2) {
                    bool cut = false;   // e ends with part of index k: the next pass goes on there
                    for (; k < p.n; ++k) {
                        const int d = side ? p.perm[k] : k;
                        if (c.t[d] > 1 || d == c.sa || d == c.sb) continue;
                        const int64_t room = quotient(most, std::max(c.nua, c.nub)), size = p.dim[d].size;
                        if (room < 2) break;
                        const int64_t pieces = ceiling(size, room);
                        e = c;
                        e.t[d] = int(ceiling(size, pieces));
                        const bool fits = box_of(p, &e);
                        if (pieces > 1) {
                            cut = fits;
                            break;
                        }
                        if (!fits) k = p.n;
                        else c = e;
                    }
                    if (cut) f(e);
                    else if (c.volume > b.volume) f(c);
                }
            }
        }
}

// Where half a wavefront's first units of a full box lie in LDS, element by
// element (those that are put, then those that are gathered): the run of A
// and the place in it.  Layouts differ in the distance between runs and in the
// skew only, so the kernel's offsets are taken once, with runs a power of two
// apart.
constexpr int kLanes = 32;
struct BankLanes {
    int n;                           // elements of a lane
    int run[8][kLanes], in[8][kLanes];
};
template <int UA, int UB>
void bank_lanes(const BoxShape& s, int log, BankLanes* out) {
    const BoxCoord c{0, 0, s.tA, s.tB, s.tC};
    out->n = UA + UB;
    for (int lane = 0; lane < kLanes; ++lane) {
        BoxUnits<UA, UB, 1> u;
        u.init(s, lane, c);
        for (int j = 0; j < UA + UB; ++j) {
            const int l = j < UA ? u.put(0, j) : u.gather(0, j - UA);
            out->run[j][lane] = l >> log;
            out->in[j][lane] = l & ((1 << log) - 1);
        }
    }
}

// LDS cycles of these accesses: a bank serves one word a cycle, 32 words in
// all.  `aligned`: the first `put` elements go as whole units, 8 lanes a cycle.
// Counts up to `limit`.
int bank_cycles(const BankLanes& lanes, int pitch, int skew, bool aligned, int put, int elem, int limit) {
    const int words = elem / 4, group = 32 / words;   // lanes served together
    int cycles = aligned ? kLanes / 8 : 0;
    for (int j = aligned ? put : 0; j < lanes.n && cycles < limit; ++j)
        for (int g = 0; g < kLanes; g += group) {
            int seen[32][32], n[32] = {}, most = 1;
            for (int lane = g; lane < g + group; ++lane) {
                int l = lanes.run[j][lane] * pitch + lanes.in[j][lane];
                l += l >> skew;
                const int bank = l * words % 32;
                bool again = false;   // the same element: one access
                for (int k = 0; k < n[bank]; ++k) again |= seen[bank][k] == l;
                if (!again) seen[bank][n[bank]++] = l;
                most = std::max(most, n[bank]);
            }
            cycles += most;
        }
    return cycles;
}

// The LDS layout: A's runs one after the other, with the distance between them
// (whole units, or an odd number of elements) and the skew that cost the
// fewest cycles; false if none fits into `cap` elements.
bool place(const Problem& p, const Box& b, int cap, BoxShape* s) {
    const int ea = elem_bytes(p.dtype_a), eb = elem_bytes(p.dtype), UA = 16 / ea, UB = 16 / eb;
    const int shift = eb == 4 ? 5 : eb == 8 ? 4 : 3;
    auto lay_out = [&](int pitch) {
        int ls[kMaxDims], at = 1;
        for (int d = 0; d < p.n; ++d) {
            if (d == b.in_run_a) at = pitch;
            ls[d] = at;
            at *= b.t[d];
        }
        for (int k = 0, d = 0; d < p.n; ++d)
            if (b.t[d] > 1 || d == b.sa || d == b.sb) s->dA[k++].ls = ls[d];
        for (int k = 0, q = 0; q < p.n; ++q) {
            const int d = p.perm[q];
            if (b.t[d] > 1 || d == b.sa || d == b.sb) s->dB[k++].ls = ls[d];
        }
    };
    int log = 0;
    while ((1 << log) < b.LA) ++log;
    lay_out(1 << log);
    s->skew = 31;
    BankLanes lanes;
    if (ea == eb)
        eb == 4 ? bank_lanes<4, 4>(*s, log, &lanes) : eb == 8 ? bank_lanes<2, 2>(*s, log, &lanes) : bank_lanes<1, 1>(*s, log, &lanes);
    else if (ea < eb)
        eb == 8 ? bank_lanes<4, 2>(*s, log, &lanes) : bank_lanes<2, 1>(*s, log, &lanes);
    else
        eb == 4 ? bank_lanes<2, 4>(*s, log, &lanes) : bank_lanes<1, 2>(*s, log, &lanes);
    const int fewest = (UA + UB) * eb / 4;   // single elements without conflicts
    int best = 1 << 30, chosen = 0;
    for (int option = 0; option < 4; ++option) {
        const bool units = option == 0;
        const int extra = option < 2 ? 0 : 12;   // a skew costs instructions too
        if (units && b.LA % UA) continue;
        if (best <= fewest + extra) break;       // what follows is no better
        const int odd = units ? UA : 1;
        const int pitch = option == 2 ? b.LA : (b.LA / odd) % 2 ? b.LA : b.LA + odd;
        const int skew = option < 2 ? 31 : shift, last = b.volume / b.LA * pitch + UA;
        if (last + (last >> skew) > cap) continue;
        const bool aligned = units && ea == eb;
        const int cycles = bank_cycles(lanes, pitch, skew, aligned, UA, eb, best - extra) + extra;
        if (cycles >= best) continue;
        best = cycles;
        chosen = pitch;
        s->aligned = aligned;
        s->skew = skew;
    }
    lay_out(chosen);
    return best < (1 << 30);
}

bool make_box(const Problem& p, bool beta0, const Box& b, BoxPlan* out) {
    const int UA = 16 / elem_bytes(p.dtype_a);
    const int* t = b.t;
    const int64_t LA = b.LA, LB = b.LB;
    const int sa = b.sa, sb = b.sb, in_run_a = b.in_run_a, in_run_b = b.in_run_b;
    BoxShape& s = out->s;
    std::memset(&s, 0, sizeof(s));
    out->units = small_box(p, b) ? 2 : 4;
    // Nontemporal stores where B is only written, in whole lines, and is a good
    // part of the 256 MiB that the last cache holds: 0.74 to 0.95 of the time on
    // six such problems (4D f32 reversal 89.4 -> 80.6 us).  With partial lines
    // they took up to 1.5 times as long, below 8 us 1.04, with beta != 0 the same.
    out->nt = beta0 && whole_lines_b(p, b) && p.extent_b >= int64_t(64) << 20;
    s.tA = sa >= 0 ? int(t[sa]) : 1;
    s.tB = sb >= 0 ? int(t[sb]) : 1;
    s.tC = b.sc >= 0 ? int(t[b.sc]) : 1;
    s.wA = int(LA / s.tA);
    s.wB = int(LB / s.tB);
    auto put = [&](BoxDim* dims, int* n, int d) {
        BoxDim& x = dims[(*n)++];
        x.ext = int(t[d]);
        x.split = (d == sa ? 1 : 0) | (d == sb ? 2 : 0) | (d == b.sc ? 4 : 0);
        x.sa = int(p.dim[d].sa);
        x.sb = int(p.dim[d].sb);
    };
    s.skew = 31;
    // a split index stays listed also where its box extent is 1
    for (int d = 0; d < p.n; ++d) {
        if (t[d] == 1 && d != sa && d != sb) continue;
        put(s.dA, &s.nA, d);
        if (d < in_run_a) s.nAr = s.nA;
    }
    for (int k = 0; k < p.n; ++k) {
        const int d = p.perm[k];
        if (t[d] == 1 && d != sa && d != sb) continue;
        put(s.dB, &s.nB, d);
        if (k < in_run_b) s.nBr = s.nB;
    }
    // grid: indices with more than one step, in B's order, so that B is written
    // as nearly one line after the other as the boxes allow
    uint64_t tiles = 1;
    for (int k = 0; k < p.n; ++k) {
        const int d = p.perm[k];
        if (t[d] == p.dim[d].size) continue;
        if (s.ng == kBoxSteps) return false;
        const uint64_t cnt = uint64_t(steps_of(p, b, d));
        tiles *= cnt;
        if (tiles >= (uint64_t(1) << 23)) return false;   // workgroups of one launch
        BoxStep& g = s.g[s.ng++];
        g.dv.init(uint32_t(cnt));
        g.sa = uint32_t(t[d] * p.dim[d].sa);
        g.sb = uint32_t(t[d] * p.dim[d].sb);
        g.split = (d == sa ? 1 : 0) | (d == sb ? 2 : 0) | (d == b.sc ? 4 : 0);
    }
    s.ntiles = uint32_t(tiles);
    s.chunk = tiles >= 1024 ? 5 : 0;
    s.sizeA = sa >= 0 ? int(p.dim[sa].size) : 1;
    s.sizeB = sb >= 0 ? int(p.dim[sb].size) : 1;
    s.sizeC = b.sc >= 0 ? int(p.dim[b.sc].size) : 1;
    return s.nA <= kBoxDims && s.nB <= kBoxDims && place(p, b, box_lds(elem_bytes(p.dtype), out->units), &s);
}

}  // namespace

bool plan_box(const Problem& p, bool beta0, BoxPlan* out, bool batched) {
    if (p.family != TTX_FAMILY_MOVED && p.family != TTX_FAMILY_PRESERVED &&
        !(batched && p.family == TTX_FAMILY_FLAT))
        return false;
    if (p.dim[0].sa != 1 || p.dim[p.perm[0]].sb != 1) return false;
    // offsets inside a box are unsigned 32-bit byte offsets
    if (p.extent_a >= (int64_t(1) << 32) || p.extent_b >= (int64_t(1) << 32)) return false;
    Box best;
    double least = 1e300;
    each_box(p, [&](const Box& b) {
        if (batched && !small_box(p, b)) return;
        const double c = box_cost(p, beta0, b);
        if (c < least) least = c, best = b;
    });
    // far from a copy's time (single elements in every run): the menu's tiles
    const double bytes = double(p.elements) * (elem_bytes(p.dtype_a) + elem_bytes(p.dtype) * (beta0 ? 1 : 2));
    return least < 4.0 * bytes / 6e6 + 10.0 && make_box(p, beta0, best, out);
}

}  // namespace ttx
