// Direct tensor contraction (Sec. 1, Sec. 4): C <- alpha * sum A*B + beta*C in
// one kernel that reads the operands and writes C where they lie.  The
// transpositions of the transpose-transpose-GEMM-transpose form become
// address arithmetic: a label group (rows, columns, contracted) is one index
// whose digits carry the strides of the two tensors that hold them.
//
// X is the operand whose free labels hold C's stride-1 label (the product's
// rows), Y the other one (columns).
#pragma once

#include <cstdint>

#include "device_types.h"

namespace ttx {

// One digit of a label group's index: its size and its strides in the two
// tensors that carry the group.  A label cut in two (a chunk walked early and
// the rest) is two digits that share a guard: the label's position is the sum
// of digit * weight over them and has to stay below guard_ext[guard].
struct ContractDigit {
    FastDiv dv;
    int guard;          // 0, 1: index into guard_ext; -1: none
    int64_t size;
    int64_t weight;
    int64_t s0, s1;
};

constexpr int kContractDigits = kMaxDims + 2;   // two labels at most are cut

struct ContractGroup {
    int nd;
    int wide;           // the index does not fit 32 bits: 64-bit divisions
    int64_t total;      // product of the digit sizes (guarded positions included)
    int64_t guard_ext[2];
    ContractDigit d[kContractDigits];

    // Offsets of index i in the group's two tensors; false past the end and
    // where a cut label's position is beyond its extent.
    __host__ __device__ __forceinline__ bool offsets(int64_t i, int64_t* o0, int64_t* o1) const {
        *o0 = *o1 = 0;
        if (i >= total) return false;
        int64_t pos0 = 0, pos1 = 0;
        if (!wide) {
            uint32_t rem = uint32_t(i);
            for (int k = 0; k < nd; ++k) {
                const ContractDigit& g = d[k];
                const uint32_t q = g.dv.div(rem), r = rem - q * g.dv.d;
                rem = q;
                *o0 += int64_t(r) * g.s0;
                *o1 += int64_t(r) * g.s1;
                if (g.guard == 0) pos0 += int64_t(r) * g.weight;
                if (g.guard == 1) pos1 += int64_t(r) * g.weight;
            }
        } else {
            uint64_t rem = uint64_t(i);
            for (int k = 0; k < nd; ++k) {
                const ContractDigit& g = d[k];
                const uint64_t q = rem / uint64_t(g.size), r = rem - q * uint64_t(g.size);
                rem = q;
                *o0 += int64_t(r) * g.s0;
                *o1 += int64_t(r) * g.s1;
                if (g.guard == 0) pos0 += int64_t(r) * g.weight;
                if (g.guard == 1) pos1 += int64_t(r) * g.weight;
            }
        }
        return pos0 < guard_ext[0] && pos1 < guard_ext[1];
    }
};

// Arguments of the contraction kernel but for pointers and scalars.
struct ContractArgs {
    ContractGroup m;    // rows: s0 in X, s1 in C
    ContractGroup n;    // columns: s0 in Y, s1 in C
    ContractGroup k;    // contracted: s0 in X, s1 in Y
    int64_t tiles_m, tiles_n;
    int64_t steps;      // k steps of a tile
    int64_t split_steps;   // and of one of its splits
    FastDiv dv_m, dv_tiles;   // by tiles_m, by tiles_m * tiles_n
    int rows;           // rows of a tile in use (<= the tile's MT)
    int walk_x, walk_y; // X's loads walk a tile's rows x + walk_x*(y + walk_y*r) -> row y + walk_y*(x + walk_x*r)
    int kwalk_x, kwalk_y;   // Y's loads walk k the same way (1: as stored)
    // C's walk in kernels that C's traffic bounds: dv_run.d rows, then the
    // columns in NT / c_cut groups (dv_cut.d) of c_cut, the groups first
    FastDiv dv_run, dv_cut;
    int c_cut;
    uint32_t first;     // the launch's first workgroup (set by the launch)
};

// Workgroups of one launch: one of 2^32 work items and more is refused.
constexpr int64_t kContractGroups = int64_t(1) << 23;

// Tile shapes: 4 waves of 16*mb rows each, 16*nb columns.
struct ContractVariant {
    int mb, nb;
};
#define TTX_CONTRACT_MENU(X) X(0, 1, 1) X(1, 1, 2) X(2, 1, 4) X(3, 1, 5) X(4, 2, 4)
constexpr int kContractVariants = 5;

// k values of one step: enough matrix instructions between two barriers to
// cover the next step's loads, in 8 to 37 KB of LDS.
constexpr int contract_kt(int elem, int mb) { return (elem == 4 ? 32 : 16) / mb; }

// Tile shapes with a kernel for sums of one step.
constexpr bool contract_has_short(int elem, int mb, int nb) { return nb == 4 && (mb == 1 || elem == 4); }

struct ContractPlan {
    int dtype = 0;
    int variant = 0;
    bool swapped = false;      // X is B
    bool xk = false, yk = false;   // X's (Y's) stride-1 label is contracted: its loads run along k
    bool vec_xy = false;   // every 16 bytes of X's and Y's walks lie in one run
    bool vec_c = false;    // and every four rows of C
    int splits = 1;
    bool packed = false;   // short sums: the operands are packed into whole tiles first
    ContractArgs args;
};

// Labels of one contraction after validation: extents and strides (in
// elements; 0 where a tensor does not carry the label).
struct ContractLabel {
    int64_t size, sa, sb, sc;
};
// Chooses roles, digit orders, tile shape and k splits (host only).  ws_elems:
// workspace elements available for the partial sums of k splits.
void plan_contraction(int dtype, const ContractLabel* labels, int count, int64_t ws_elems, ContractPlan* out);
// The same with the tile shape, the k splits and the packing given (timing).
void plan_contraction_as(int dtype, const ContractLabel* labels, int count, int variant, int splits, bool packed,
                         ContractPlan* out);

hipError_t launch_contraction(const ContractPlan& p, const void* A, const void* B, void* C, void* workspace,
                              double alpha, double beta, hipStream_t stream);
hipError_t launch_contract_f32(const ContractPlan& p, const float* X, const float* Y, float* C, float* part,
                               float alpha, float beta, hipStream_t stream);
hipError_t launch_contract_f64(const ContractPlan& p, const double* X, const double* Y, double* C, double* part,
                               double alpha, double beta, hipStream_t stream);

}  // namespace ttx
