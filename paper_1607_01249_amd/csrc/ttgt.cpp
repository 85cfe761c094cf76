// Tensor contraction in its transpose-transpose-GEMM-transpose form (Sec. 1:
// a contraction cast as a matrix product through transpositions; Sec. 4: the
// transposition as the building block of a contraction compiler).
//
// Planning (host only) splits the labels into the product's rows (A's free
// labels), columns (B's free labels) and the contracted labels, and describes
// the matrix form: an operand whose free and contracted labels form two
// contiguous blocks is already a matrix (packed with the left- or
// right-operand panel kind, whichever reads it in storage order, since both
// kinds produce the same panel layout), provided both operands use one
// contracted order.  Execution folds the transpositions and the packing into
// the addresses of one kernel (contract.h), which writes alpha * product +
// beta * C in C's mode order (Eqn. 1).  On an MI355X, against the chain of
// transpositions, packings, panel GEMM and transposition of the product that
// it replaces: m = n = k = 1600 FP32 147 -> 82 us; a 24^6 result from a sum of
// 16 (FP32, beta != 0) 650 -> 310 us, since the 729 MiB product is neither
// written nor read back; 96 x 64 x 512 from a sum of 8 (FP64) 36 -> 13 us, one
// launch instead of five; small ones of 26 to 40 us in 7 to 8.
#include <algorithm>
#include <cstring>
#include <memory>
#include <vector>

#include "contract.h"
#include "ttx_internal.h"

struct ttx_contraction {
    int dtype = TTX_F32, panel = 16;
    int64_t m = 1, n = 1, k = 1;
    int64_t bytes_a = 0, bytes_b = 0, bytes_c = 0;     // byte extents of A, B, C
    bool trans_a = false, trans_b = false;
    int kind_a = TTX_PACK_MFMA_A, kind_b = TTX_PACK_MFMA_B;
    int64_t ws = 0;                    // workspace bytes
    std::vector<int> ord_m, ord_n, ord_k;
    ttx::ContractPlan plan;
};

namespace ttx {
namespace {

// 1: `labels` is block X then block Y; 2: block Y then block X; 0: neither.
// X and Y hold the tensor's labels of each group in its own order.
int block_layout(const std::vector<int>& labels, const std::vector<int>& X, const std::vector<int>& Y) {
    std::vector<int> xy(X), yx(Y);
    xy.insert(xy.end(), Y.begin(), Y.end());
    yx.insert(yx.end(), X.begin(), X.end());
    if (labels == xy) return 1;
    if (labels == yx) return 2;
    return 0;
}

// Product of the labels' extents; -1 when it does not fit in int64_t.
int64_t product(const std::vector<int>& labels, const std::vector<std::pair<int, int64_t>>& ext) {
    int64_t p = 1;
    for (int l : labels)
        for (const auto& e : ext)
            if (e.first == l && __builtin_mul_overflow(p, e.second, &p)) return -1;
    return p;
}

int64_t extent_of(int l, const std::vector<std::pair<int, int64_t>>& ext) {
    for (const auto& e : ext)
        if (e.first == l) return e.second;
    return 1;
}

int64_t align256(int64_t x) { return (x + 255) / 256 * 256; }

bool overlaps(const void* p, int64_t pn, const void* q, int64_t qn) {
    if (pn <= 0 || qn <= 0) return false;
    const uintptr_t a = reinterpret_cast<uintptr_t>(p), b = reinterpret_cast<uintptr_t>(q);
    return a < b + uint64_t(qn) && b < a + uint64_t(pn);
}

}  // namespace
}  // namespace ttx

using namespace ttx;

extern "C" {

ttx_status ttx_contraction_create(ttx_contraction** plan, ttx_dtype dtype, int na, const int* labels_a,
                                  const int64_t* size_a, int nb, const int* labels_b, const int64_t* size_b,
                                  int nc, const int* labels_c, const int64_t* size_c) {
    if (!plan) return fail(TTX_EINVAL, "plan must not be NULL");
    *plan = nullptr;
    if (!dtype_valid(dtype)) return fail(TTX_EINVAL, "unknown dtype");
    if (dtype != TTX_F32 && dtype != TTX_F64)
        return fail(TTX_EUNSUPPORTED, "contraction: TTX_F32 or TTX_F64 (the matrix-core GEMM's types)");
    const int cnt[3] = {na, nb, nc};
    const int* lab[3] = {labels_a, labels_b, labels_c};
    const int64_t* siz[3] = {size_a, size_b, size_c};
    std::vector<int> L[3];
    std::vector<std::pair<int, int64_t>> ext;
    for (int t = 0; t < 3; ++t) {
        if (cnt[t] < 0 || cnt[t] > TTX_MAX_DIMS) return fail(TTX_EINVAL, "mode count outside 0..TTX_MAX_DIMS");
        if (cnt[t] > 0 && (!lab[t] || !siz[t])) return fail(TTX_EINVAL, "NULL labels or extents");
        for (int d = 0; d < cnt[t]; ++d) {
            const int l = lab[t][d];
            const int64_t s = siz[t][d];
            if (s < 0) return fail(TTX_EINVAL, "negative extent");
            if (std::find(L[t].begin(), L[t].end(), l) != L[t].end())
                return fail(TTX_EINVAL, "a tensor carries a label twice");
            L[t].push_back(l);
            bool seen = false;
            for (const auto& e : ext)
                if (e.first == l) {
                    seen = true;
                    if (e.second != s) return fail(TTX_EINVAL, "a label has two extents");
                }
            if (!seen) ext.push_back({l, s});
        }
    }
    auto has = [&](int t, int l) { return std::find(L[t].begin(), L[t].end(), l) != L[t].end(); };
    for (const auto& e : ext) {
        const int c = has(0, e.first) + has(1, e.first) + has(2, e.first);
        if (c == 3) return fail(TTX_EINVAL, "batch label (carried by A, B and C)");
        if (c != 2) return fail(TTX_EINVAL, "a label is carried by one tensor only");
    }
    for (int t = 0; t < 3; ++t)
        if (product(L[t], ext) < 0 || product(L[t], ext) > (int64_t(1) << 56))
            return fail(TTX_EINVAL, "tensor too large");
    std::unique_ptr<ttx_contraction> p(new ttx_contraction);
    p->dtype = dtype;
    // groups, each in its own tensor's order
    std::vector<int> Ma, Ka, Kb, Nb;
    for (int l : L[0]) (has(2, l) ? Ma : Ka).push_back(l);
    for (int l : L[1]) (has(2, l) ? Nb : Kb).push_back(l);
    const int lay_a = block_layout(L[0], Ma, Ka);   // 1: (M, K), 2: (K, M)
    const int lay_b = block_layout(L[1], Kb, Nb);   // 1: (K, N), 2: (N, K)
    std::vector<int> K;
    if (lay_a && lay_b && Ka == Kb) {
        K = Ka;
    } else if (lay_a && lay_b) {   // both matrices, contracted orders differ: transpose the smaller
        const bool a_smaller = product(L[0], ext) <= product(L[1], ext);
        K = a_smaller ? Kb : Ka;
        (a_smaller ? p->trans_a : p->trans_b) = true;
    } else if (lay_a) {
        K = Ka;
        p->trans_b = true;
    } else if (lay_b) {
        K = Kb;
        p->trans_a = true;
    } else {
        K = Ka;
        p->trans_a = p->trans_b = true;
    }
    if (!p->trans_b && Kb != K) p->trans_b = true;
    if (!p->trans_a && Ka != K) p->trans_a = true;
    p->ord_m = Ma;
    p->ord_n = Nb;
    p->ord_k = K;
    p->m = product(Ma, ext);
    p->n = product(Nb, ext);
    p->k = product(K, ext);
    const int64_t es = elem_bytes(dtype);
    p->bytes_a = product(L[0], ext) * es;
    p->bytes_b = product(L[1], ext) * es;
    p->bytes_c = product(L[2], ext) * es;
    p->panel = (dtype == TTX_F32 && p->m >= 32 && p->n >= 32) ? 32 : 16;
    // how a packing step would read each operand: a right-operand kind reads a
    // (contracted, free) matrix in its storage order, a left-operand kind a (free, contracted) one
    p->kind_a = (p->trans_a || lay_a == 1) ? TTX_PACK_MFMA_A : TTX_PACK_MFMA_B;
    p->kind_b = (p->trans_b || lay_b == 1) ? TTX_PACK_MFMA_B : TTX_PACK_MFMA_A;
    // workspace: what the matrix form needs at most (operand matrices where
    // transposed, panels, product); the partial sums of a cut sum fit in it
    const int64_t kb = 64 / p->panel, Kp = (p->k + kb - 1) / kb * kb;
    const int64_t mp = (p->m + p->panel - 1) / p->panel, nq = (p->n + p->panel - 1) / p->panel;
    int64_t off = 0;
    auto take = [&](int64_t elems) { off += align256(elems * es); };
    if (p->trans_a) take(p->m * p->k);
    if (p->trans_b) take(p->k * p->n);
    take(mp * p->panel * Kp);
    take(nq * p->panel * Kp);
    take(p->m * p->n);
    p->ws = (p->m == 0 || p->n == 0) ? 0 : off;
    if (p->ws) {
        std::vector<ContractLabel> labs;
        for (const auto& e : ext) {
            ContractLabel l{e.second, 0, 0, 0};
            int64_t* const stride[3] = {&l.sa, &l.sb, &l.sc};
            for (int t = 0; t < 3; ++t) {
                int64_t at = 1;
                for (int x : L[t]) {
                    if (x == e.first) *stride[t] = at;
                    at *= std::max<int64_t>(extent_of(x, ext), 1);
                }
            }
            labs.push_back(l);
        }
        plan_contraction(dtype, labs.data(), int(labs.size()), p->ws / es, &p->plan);
    }
    *plan = p.release();
    return TTX_OK;
}

ttx_status ttx_contraction_describe(const ttx_contraction* plan, ttx_contraction_info* info) {
    if (!plan || !info) return fail(TTX_EINVAL, "NULL argument");
    std::memset(info, 0, sizeof(*info));
    info->m = plan->m;
    info->n = plan->n;
    info->k = plan->k;
    info->panel = plan->panel;
    info->transposed_a = plan->trans_a;
    info->transposed_b = plan->trans_b;
    info->pack_kind_a = plan->kind_a;
    info->pack_kind_b = plan->kind_b;
    info->n_m = int(plan->ord_m.size());
    info->n_n = int(plan->ord_n.size());
    info->n_k = int(plan->ord_k.size());
    std::copy(plan->ord_m.begin(), plan->ord_m.end(), info->order_m);
    std::copy(plan->ord_n.begin(), plan->ord_n.end(), info->order_n);
    std::copy(plan->ord_k.begin(), plan->ord_k.end(), info->order_k);
    info->workspace_bytes = plan->ws;
    return TTX_OK;
}

ttx_status ttx_contraction_execute(const ttx_contraction* plan, double alpha, const void* A, const void* B,
                                   double beta, void* C, void* workspace, hipStream_t stream) {
    if (!plan) return fail(TTX_EINVAL, "plan must not be NULL");
    if (plan->m == 0 || plan->n == 0) return TTX_OK;   // C is empty
    if ((plan->bytes_a && !A) || (plan->bytes_b && !B) || !C || !workspace)
        return fail(TTX_EINVAL, "NULL tensor or workspace pointer");
    const uintptr_t es = uintptr_t(elem_bytes(plan->dtype));
    if (reinterpret_cast<uintptr_t>(A) % es || reinterpret_cast<uintptr_t>(B) % es ||
        reinterpret_cast<uintptr_t>(C) % es || reinterpret_cast<uintptr_t>(workspace) % es)
        return fail(TTX_EINVAL, "pointer not aligned to the element size");
    if (overlaps(C, plan->bytes_c, A, plan->bytes_a) || overlaps(C, plan->bytes_c, B, plan->bytes_b))
        return fail(TTX_EOVERLAP, "C overlaps an operand");
    if (overlaps(workspace, plan->ws, A, plan->bytes_a) || overlaps(workspace, plan->ws, B, plan->bytes_b) ||
        overlaps(workspace, plan->ws, C, plan->bytes_c))
        return fail(TTX_EOVERLAP, "the workspace overlaps a tensor");
    const hipError_t e = launch_contraction(plan->plan, A, B, C, workspace, alpha, beta, stream);
    return e == hipSuccess ? TTX_OK : fail(TTX_EHIP, std::string("kernel launch: ") + hipGetErrorString(e));
}

ttx_status ttx_contraction_destroy(ttx_contraction* plan) {
    delete plan;
    return TTX_OK;
}

}  // extern "C"
