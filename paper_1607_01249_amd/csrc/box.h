// Box tiles: a tile is a box over the merged indices that holds whole runs of
// A and whole runs of B, moved in 16-byte units on both sides.
//
// A's run is A's first indices, whole, up to one that is cut (split A); B's run
// likewise in B's order (split B, possibly the same index).  Where these alone
// would leave a box small, a third index fills it (whole or cut); every other
// index has extent 1 in the box.  The box is read run by run into LDS in A's order
// and written run by run in B's order, each unit gathered from LDS.  Where
// each unit lies (offsets in A, B and LDS) is worked out once per workgroup
// and box shape and serves every tile of that shape; boxes cut short by the
// end of a split index are another shape.  A run whose length is not a whole
// number of units ends with a unit that overlaps the one before it.
#pragma once

#ifndef __HIPCC_RTC__
#include <cstdint>
#endif

#include "device_types.h"

namespace ttx {

constexpr int kBoxDims = 6;     // indices of extent > 1 in a box
constexpr int kBoxSteps = 8;    // indices of the grid of boxes
constexpr int kBoxUnits = 4;    // most units per thread and side

// Whether B starts on a 128-byte line.  Nontemporal stores of partial lines
// are slow, and a B that does not has them throughout.
inline bool box_on_line(const void* B) { return (unsigned long long)(B) % 128 == 0; }

struct BoxDim {
    int ext;         // extent in the box
    int split;       // 1: split A, 2: split B, 3: both, 4: fill
    int sa, sb;      // element strides in A and B
    int ls;          // stride in the LDS box
};

// One index of the grid of boxes.
struct BoxStep {
    FastDiv dv;      // boxes along it
    uint32_t sa, sb; // elements from one box to the next in A and B
    int split;       // as in BoxDim
};

// The type-independent arguments of a box kernel.
struct BoxShape {
    uint32_t ntiles;
    int chunk;           // log2 of the boxes in a row that one XCD takes
    int ng;              // grid indices
    int tA, tB, tC;      // box extents of split A, split B and fill (1 where there is none)
    int sizeA, sizeB, sizeC;   // and their full extents
    int nA, nAr, nB, nBr;   // dims in A's order, of these in A's run; in B's order
    int wA, wB;          // elements of a run per step of its split index
    int aligned;         // A's runs start on whole units in LDS, and lie there as they are
    int skew;            // element l of the box lies at l + (l >> skew) in LDS (31: at l)
    BoxDim dA[kBoxDims], dB[kBoxDims];
    BoxStep g[kBoxSteps];
};

// Where a box lies and how far it extends along the indices that it cuts.
struct BoxCoord {
    uint32_t oa, ob;
    int ea, eb, ec;
};
__host__ __device__ __forceinline__ BoxCoord box_coord(const BoxShape& s, uint32_t t) {
    BoxCoord c{0, 0, s.tA, s.tB, s.tC};
    for (int q = 0; q < s.ng; ++q) {
        const BoxStep g = s.g[q];
        const uint32_t next = g.dv.div(t), r = t - next * g.dv.d;
        t = next;
        c.oa += r * g.sa;
        c.ob += r * g.sb;
        if ((g.split & 1) && s.sizeA - int(r) * s.tA < s.tA) c.ea = s.sizeA - int(r) * s.tA;
        if ((g.split & 2) && s.sizeB - int(r) * s.tB < s.tB) c.eb = s.sizeB - int(r) * s.tB;
        if ((g.split & 4) && s.sizeC - int(r) * s.tC < s.tC) c.ec = s.sizeC - int(r) * s.tC;
    }
    return c;
}

// v / ext for v < 2^20: the quotient of v + 1/2 lies at least 1 / (2 ext) from
// a whole number, and two roundings and a reciprocal good to 2^-22 move it by
// less than v 2^-21 / ext.
__host__ __device__ __forceinline__ float box_inverse(int ext) {
#ifdef __HIP_DEVICE_COMPILE__
    return __builtin_amdgcn_rcpf(float(ext));
#else
    return 1.0f / float(ext);
#endif
}
__host__ __device__ __forceinline__ int box_quotient(int v, float inverse) {
    return int((float(v) + 0.5f) * inverse);
}

// Units of one thread for boxes of one shape.  The indices are the outer loop
// and the units the inner one: an index's constants are read once.
template <int UA, int UB, int NU = kBoxUnits>
struct BoxUnits {
    int nua, nub;                   // units of the whole box
    int skew;
    bool whole_a;                   // A's runs are whole units (aligned in LDS)
    bool shorter;                   // a run is shorter than a unit: element by element
    int rel_a[NU], rel_b[NU];
    int lds_a[NU];
    uint32_t lds_b[NU][(UB + 1) / 2];   // two offsets a word

    __host__ __device__ __forceinline__ static int extent(const BoxDim& d, const BoxCoord& c) {
        return (d.split & 1) ? c.ea : (d.split & 2) ? c.eb : d.split ? c.ec : d.ext;
    }
    // LDS element j of unit i: of A's (before the skew), of B's
    __host__ __device__ __forceinline__ int put(int i, int j) const { return lds_a[i] + j; }
    __host__ __device__ __forceinline__ int gather(int i, int j) const {
        return UB == 1 ? int(lds_b[i][0]) : int((lds_b[i][j / 2] >> (j % 2 * 16)) & 0xffffu);
    }

    __host__ __device__ __forceinline__ void init(const BoxShape& s, int tid, const BoxCoord& c) {
        const int LA = s.wA * c.ea, LB = s.wB * c.eb;
        shorter = LA < UA || LB < UB;
        if (shorter) return;
        whole_a = s.aligned && LA % UA == 0;
        skew = s.skew;
        const int ua = (LA + UA - 1) / UA, ub = (LB + UB - 1) / UB;
        nua = ua;
        nub = ub;
        for (int k = s.nAr; k < s.nA; ++k) nua *= extent(s.dA[k], c);
        for (int k = s.nBr; k < s.nB; ++k) nub *= extent(s.dB[k], c);
        int r[NU];
        const float iua = box_inverse(ua), iub = box_inverse(ub);
#pragma unroll
        for (int i = 0; i < NU; ++i) {
            int e = tid + kThreads * i;
            if (e >= nua) e = nua - 1;   // threads past the last unit repeat it
            r[i] = box_quotient(e, iua);
            int at = (e - r[i] * ua) * UA;
            if (at > LA - UA) at = LA - UA;
            rel_a[i] = lds_a[i] = at;
        }
        for (int k = s.nAr; k < s.nA; ++k) {
            const BoxDim d = s.dA[k];
            const int ext = extent(d, c);
            const float inv = box_inverse(ext);
#pragma unroll
            for (int i = 0; i < NU; ++i) {
                const int q = box_quotient(r[i], inv), x = r[i] - q * ext;
                r[i] = q;
                rel_a[i] += x * d.sa;
                lds_a[i] += x * d.ls;
            }
        }
        int l[NU], at[NU];
#pragma unroll
        for (int i = 0; i < NU; ++i) {
            int e = tid + kThreads * i;
            if (e >= nub) e = nub - 1;
            r[i] = box_quotient(e, iub);
            at[i] = (e - r[i] * ub) * UB;
            if (at[i] > LB - UB) at[i] = LB - UB;
            rel_b[i] = at[i];
            l[i] = 0;
        }
        for (int k = s.nBr; k < s.nB; ++k) {
            const BoxDim d = s.dB[k];
            const int ext = extent(d, c);
            const float inv = box_inverse(ext);
#pragma unroll
            for (int i = 0; i < NU; ++i) {
                const int q = box_quotient(r[i], inv), x = r[i] - q * ext;
                r[i] = q;
                rel_b[i] += x * d.sb;
                l[i] += x * d.ls;
            }
        }
        // the lanes of a unit, along B's run
        int v[NU][UB], g[NU][UB];
#pragma unroll
        for (int i = 0; i < NU; ++i)
#pragma unroll
            for (int j = 0; j < UB; ++j) {
                v[i][j] = at[i] + j;
                g[i][j] = l[i];
            }
        for (int k = 0; k + 1 < s.nBr; ++k) {
            const BoxDim d = s.dB[k];
            const float inv = box_inverse(d.ext);
#pragma unroll
            for (int i = 0; i < NU; ++i)
#pragma unroll
                for (int j = 0; j < UB; ++j) {
                    const int q = box_quotient(v[i][j], inv);
                    g[i][j] += (v[i][j] - q * d.ext) * d.ls;
                    v[i][j] = q;
                }
        }
        const int ls = s.dB[s.nBr - 1].ls;   // the last (split) index takes the rest
#pragma unroll
        for (int i = 0; i < NU; ++i)
#pragma unroll
            for (int j = 0; j < UB; ++j) {
                const uint32_t x = uint32_t(g[i][j] + v[i][j] * ls);
                if (j % 2 == 0) lds_b[i][j / 2] = x;
                else lds_b[i][j / 2] |= x << 16;
            }
        if (skew < 31) {
            const uint32_t low = (1u << (16 - skew)) - 1;
#pragma unroll
            for (int i = 0; i < NU; ++i)
#pragma unroll
                for (int j = 0; j < (UB + 1) / 2; ++j)
                    lds_b[i][j] += lds_b[i][j] >> skew & (low << 16 | low);
        }
    }
};

template <typename T, typename S = T>
struct BoxPtrs {
    const S* A;
    const T* Bsrc;
    T* Bdst;
    T alpha, beta;
};
template <typename T, typename S = T>
struct BoxArgs : BoxShape, BoxPtrs<T, S> {};

// LDS elements of a box of B's type: 4 KiB per unit and thread, and room for
// the padding of its runs.
constexpr int box_lds(int elem, int units) { return (4096 * units + 1024 * units) / elem; }

// One problem of a launch over many (FP32 and FP64).
struct BoxBatchDesc {
    union {
        BoxArgs<float> f32;
        BoxArgs<double> f64;
    };
    int kind;            // f32 beta, f32 beta == 0, f64 beta, f64 beta == 0
    __host__ __device__ BoxBatchDesc() {}
};
constexpr int kBoxBuckets = 1024;
struct BoxBatchGrid {
    uint32_t grid;       // workgroups
    uint32_t chunks;     // of 2^chunk boxes
    int chunk, shift;    // a bucket covers 2^shift chunks
};

// A box for one problem (host).
struct BoxPlan {
    BoxShape s;
    int units;           // per thread and side that hold the box: 2 or 4
    bool nt;             // nontemporal stores, if B starts on a line
};
// The best box for a problem, false if it has none (no contiguous runs of a
// unit on both sides, offsets beyond 32 bits, empty problems).  `batched`: for
// a launch over many problems (two units a thread, and flat problems too,
// which otherwise have kernels of their own).
struct Problem;
bool plan_box(const Problem& p, bool beta0, BoxPlan* out, bool batched = false);

}  // namespace ttx
