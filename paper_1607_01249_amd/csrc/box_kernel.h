// The box-tile kernel (see box.h).
//
// Large problems are bound by memory: whole runs on both sides reach 5.5 TB/s
// (6D f64 [20,16,16,20,16,16], update, 0.117 ms; the whole-unit dense tiles
// took 0.175) and short or unaligned ones 4.6 to 5.4 (4D f32 reversal 0.080 ms
// with nontemporal stores, 6D f32 reversal with odd extents 0.136), where a copy
// runs at 6.1.  Small ones
// are bound by one box's chain: arguments, offsets, loads, LDS, stores.  The
// offsets were the bound at first: with integer divisions and one pass of the
// indices per unit a box cost 1000 instructions and 80 scalar loads one after
// the other, 1.35 times the menu's time over all; the indices as the outer loop
// and float quotients brought 0.98, one box per workgroup (8 wavefronts a SIMD
// where the loop left 4), 32 boxes in a row per XCD and B's order 0.81.
#pragma once

#include "box.h"
#include "tile_kernels.h"

namespace ttx {

// One tile whose runs are shorter than a unit: element by element in B's
// order, without LDS.
template <typename T, bool BETA0, typename S>
__device__ __forceinline__ void box_elements(const BoxShape& s, const BoxPtrs<T, S>& a, const BoxCoord& c) {
    int n = 1;
    for (int k = 0; k < s.nB; ++k) n *= BoxUnits<1, 1>::extent(s.dB[k], c);
    for (int e = threadIdx.x; e < n; e += kThreads) {
        uint32_t v = uint32_t(e);
        int64_t oa = c.oa, ob = c.ob;
        for (int k = 0; k < s.nB; ++k) {
            const uint32_t ext = uint32_t(BoxUnits<1, 1>::extent(s.dB[k], c)), q = v / ext, x = v - q * ext;
            v = q;
            oa += int64_t(x) * s.dB[k].sa;
            ob += int64_t(x) * s.dB[k].sb;
        }
        T b{};
        if constexpr (!BETA0) b = a.Bsrc[ob];
        a.Bdst[ob] = epilogue<T, 1, BETA0>(conv<T, S>(a.A[oa]), b, a.alpha, a.beta);
    }
}

// Workgroup b's box.  Workgroups go round the 8 XCDs; `chunk` (log2) boxes in
// a row stay on one XCD, so that the lines which neighbouring boxes share meet
// in its L2, while the XCDs together stay within 8 chunks of each other.  The
// boxes after the last full set of chunks keep their order.
__device__ __forceinline__ uint32_t box_id(uint32_t b, uint32_t n, int chunk) {
    const uint32_t set = b >> (chunk + 3);
    if (((set + 1) << (chunk + 3)) > n) return b;
    const uint32_t r = b & ((8u << chunk) - 1);
    return (set << (chunk + 3)) + ((r & 7) << chunk) + (r >> 3);
}

// A uniform base and an unsigned 32-bit byte offset: one register a lane.
template <typename E>
__device__ __forceinline__ const E* box_at(const E* base, int rel) {
    return reinterpret_cast<const E*>(reinterpret_cast<const char*>(base) + uint32_t(rel) * uint32_t(sizeof(E)));
}
template <typename E>
__device__ __forceinline__ E* box_at(E* base, int rel) {
    return reinterpret_cast<E*>(reinterpret_cast<char*>(base) + uint32_t(rel) * uint32_t(sizeof(E)));
}

// Reads a word of every 64-byte line of the arguments: they are read in
// chains of a few words each, and the first workgroups of a compute unit would
// wait for one line after the other.
template <typename Args>
__device__ __forceinline__ void touch(const Args& a) {
    const uint32_t* w = reinterpret_cast<const uint32_t*>(&a);
    constexpr int n = int(sizeof(Args) / 64) < 10 ? int(sizeof(Args) / 64) : 10;
    uint32_t x[n];
#pragma unroll
    for (int i = 0; i < n; ++i) x[i] = w[16 * i + 15];
#pragma unroll
    for (int i = 0; i < n; ++i) asm volatile("" ::"s"(x[i]));
}

// Box t.  NT: nontemporal stores.
template <typename T, typename S, bool BETA0, int NU, bool NT = false>
__device__ __forceinline__ void box_body(T* lds, const BoxShape& s, const BoxPtrs<T, S>& a, uint32_t t) {
    constexpr int UA = kVec<S>, UB = kVec<T>;
    const BoxCoord c = box_coord(s, t);
    BoxUnits<UA, UB, NU> u;
    u.init(s, threadIdx.x, c);
    if (u.shorter) return box_elements<T, BETA0, S>(s, a, c);
    const S* A = a.A + c.oa;
    vec_t<S, UA> va[NU];
    vec_t<T, UB> vb[NU];
    // every unit is loaded, also the repeats past the last one (one request a
    // wavefront): loads under a branch would each be waited for at its end
#pragma unroll
    for (int i = 0; i < NU; ++i) ld_part<S, UA>(va[i], box_at(A, u.rel_a[i]), UA);
    if constexpr (!BETA0) {
        const T* B = a.Bsrc + c.ob;
#pragma unroll
        for (int i = 0; i < NU; ++i) ld_part<T, UB>(vb[i], box_at(B, u.rel_b[i]), UB);
    }
    bool whole = false;
    if constexpr (std::is_same<T, S>::value) {
        whole = u.whole_a;
        if (whole) {
#pragma unroll
            for (int i = 0; i < NU; ++i)
                if (kThreads * i < u.nua) st<T, UB, false>(lds + u.lds_a[i], va[i]);
        }
    }
    if (!whole) {
        if (u.skew < 31) {
#pragma unroll
            for (int i = 0; i < NU; ++i)
                if (kThreads * i < u.nua) {
#pragma unroll
                    for (int j = 0; j < UA; ++j) {
                        const int l = u.put(i, j);
                        lds[l + (l >> u.skew)] = conv<T, S>(lane<S, UA>(va[i], j));
                    }
                }
        } else {
#pragma unroll
            for (int i = 0; i < NU; ++i)
                if (kThreads * i < u.nua) {
#pragma unroll
                    for (int j = 0; j < UA; ++j) lds[u.put(i, j)] = conv<T, S>(lane<S, UA>(va[i], j));
                }
        }
    }
    // overlapping units read B twice: every read ends before any store
    if constexpr (!BETA0) __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0)
    __syncthreads();
    T* B = a.Bdst + c.ob;
#pragma unroll
    for (int i = 0; i < NU; ++i)
        if (kThreads * i < u.nub) {
            vec_t<T, UB> v;
#pragma unroll
            for (int j = 0; j < UB; ++j) set_lane<T, UB>(v, j, lds[u.gather(i, j)]);
            st_part<T, UB, NT>(box_at(B, u.rel_b[i]), epilogue<T, UB, BETA0>(v, vb[i], a.alpha, a.beta), UB);
        }
}

template <typename T, typename S, bool BETA0, int NU, bool NT>
__global__ __launch_bounds__(kThreads, 5) void k_box(BoxArgs<T, S> a) {
    __shared__ __align__(16) T lds[box_lds(sizeof(T), NU)];
    touch(a);
    box_body<T, S, BETA0, NU, NT>(lds, a, a, box_id(blockIdx.x, a.ntiles, a.chunk));
}

}  // namespace ttx
