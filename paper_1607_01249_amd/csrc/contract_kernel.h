// The direct contraction kernels (see contract.h): one workgroup of four waves
// computes a tile of MT = 64*MB rows x NT = 16*NB columns of C with the
// 16 x 16 x 4 matrix instructions.
//
// Long sums (k_contract) are bound by the matrix cores: m = n = k = 1600 FP32
// runs at 100 TFLOP/s and 4096 x 4096 x 1024 at 118, of the 156 that a loop of
// these instructions alone reaches; FP64 2048 x 2048 x 1024 at 54 of 73 that a
// large library product reaches.  A wave's own instruction stream was the
// bound on the way there (one workgroup a CU, 128 x 128 tiles, 100 steps of
// 16: 152 us while each of these held): loads under a branch a lane (the
// compiler waits for each before the next), operands read from LDS right
// before their use, addresses and zero tests worked out in every step.
// Hence unconditional loads, pinned reads, two steps a trip so that the
// buffer is a constant, and k offsets computed 256 at a time.
//
// Short sums (k_contract_short) are bound by C: 24^6 FP32 results from sums of
// 16 move C at 5.0 TB/s with beta != 0 (0.310 ms; 0.48 ms before C was asked
// for ahead of the operands and walked in its own order).
#pragma once

#include <hip/hip_runtime.h>

#include "contract.h"
#include "tile_kernels.h"

namespace ttx {

// 16 x 16 x 4 products P * Q: lane l holds row frag(l % 16) of P's block and
// column l % 16 of Q's at k = l / 16, and afterwards rows 4*(l/16) .. + 3 of
// column l % 16.  (The FP64 instruction leaves register r the block's row
// l/16 + 4*r: its rows go in permuted.)
template <typename T>
struct Mma;
template <>
struct Mma<float> {
    typedef float Acc __attribute__((ext_vector_type(4)));
    __device__ static __forceinline__ Acc step(float p, float q, Acc c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(p, q, c, 0, 0, 0);
    }
    __device__ static __forceinline__ int frag(int i) { return i; }
};
template <>
struct Mma<double> {
    typedef double Acc __attribute__((ext_vector_type(4)));
    __device__ static __forceinline__ Acc step(double p, double q, Acc c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(p, q, c, 0, 0, 0);
    }
    __device__ static __forceinline__ int frag(int i) { return 4 * (i & 3) + (i >> 2); }
};

// Four consecutive elements at any element boundary, in 16-byte accesses.
template <typename T>
__device__ __forceinline__ typename Mma<T>::Acc load_rows(const T* p) {
    constexpr int U = 16 / int(sizeof(T));
    typename Mma<T>::Acc v;
#pragma unroll
    for (int q = 0; q < 4; q += U) {
        vec_t<T, U> part;
        ld_part<T, U>(part, p + q, U);
#pragma unroll
        for (int j = 0; j < U; ++j) v[q + j] = part[j];
    }
    return v;
}
template <typename T>
__device__ __forceinline__ void store_rows(T* p, typename Mma<T>::Acc v) {
    constexpr int U = 16 / int(sizeof(T));
#pragma unroll
    for (int q = 0; q < 4; q += U) {
        vec_t<T, U> part;
#pragma unroll
        for (int j = 0; j < U; ++j) part[j] = v[q + j];
        st_part<T, U, false>(p + q, part, U);
    }
}

// An operand's tile in LDS: KT x ROWS elements, rows contiguous.  Four
// consecutive k start 16 banks apart (the lanes of one operand read take four
// k of 16 rows each), and each further group of four k is moved by as many
// elements as rows that a wave of loads along k writes at once.
template <int ROWS, int PAD>
struct ContractLds {
    static constexpr int LD = (ROWS / 16) % 2 ? ROWS : ROWS + 16;
    static constexpr int LQ = 4 * LD + PAD;
    static constexpr int elems(int kt) { return kt / 4 * LQ; }
    __device__ static __forceinline__ int at(int k, int row) { return (k >> 2) * LQ + (k & 3) * LD + row; }
};

constexpr int contract_pad(int elem, int kt) { return 64 * (16 / elem) / kt; }

// Loads of one operand's tile, a step ahead in registers, U places of the walk
// along the operand's stride-1 label each (KW: contracted, the places run
// along k; else along the rows).  VEC: every U consecutive places are one run,
// one 16-byte load at element alignment; otherwise lanes take consecutive
// places, U times.  Loads are unconditional: a row that does not exist has
// the offset of row 0 and its sums are not stored; a k that does not exist is
// read at k = 0 and becomes zero, in both operands, on its way to LDS; lanes
// beyond the walk (80 columns: 20 or 40 units in a row of 32 or 64 lanes)
// read its last place, a whole unit with VEC, and store nothing.
template <typename T, int ROWS, int KT, bool KW, bool VEC>
struct ContractLoad {
    static constexpr int U = 16 / int(sizeof(T));
    static constexpr int W = (KW ? KT : ROWS) / U;        // units along the walk
    static constexpr int P = pow2_ceil(W), R = 256 / P;   // R rows (KW) or k values a pass
    static constexpr int E = KW ? ROWS : KT, N = (E + R - 1) / R;
    using L = ContractLds<ROWS, contract_pad(sizeof(T), KT)>;
    typedef T Vec __attribute__((ext_vector_type(U)));
    struct __attribute__((packed, aligned(sizeof(T)))) Loose {   // 16 bytes at any element
        Vec v;
    };
    Vec v[N];
    const char* at[KW ? N : VEC ? 1 : U];   // each pass's row, or the unit's rows
    int place[U];   // the unit's k values, or its rows in LDS
    int other;      // first row, or first k

    // rows: byte offsets of the tile's rows.  wa x wb: the walk over the first
    // `used` rows, or over k.
    __host__ __device__ __forceinline__ void init(int tid, const T* p, const int64_t* rows, int wa, int wb, int used) {
        const char* base = reinterpret_cast<const char*>(p);
        int u = tid % P;
        if (P != W && u >= W) u = W - 1;
        other = tid / P;
#pragma unroll
        for (int j = 0; j < U; ++j) {
            int r = VEC ? u * U + j : u + j * W;
            if (wa > 1 && r < used) {
                const int x = r % wa, q = r / wa;
                r = q % wb + wb * (x + wa * (q / wb));
            }
            place[j] = r;
        }
        if constexpr (KW) {
#pragma unroll
            for (int i = 0; i < N; ++i) at[i] = base + rows[other + i * R < ROWS ? other + i * R : ROWS - 1];
        } else {
#pragma unroll
            for (int j = 0; j < (VEC ? 1 : U); ++j) at[j] = base + rows[place[j]];
        }
    }
    // not a lane beyond the walk, or past the last row or k of the tile
    __device__ __forceinline__ bool live(int i) const {
        return (P == W || int(threadIdx.x) % P < W) && (E % R == 0 || other + i * R < E);
    }
    __host__ __device__ __forceinline__ int k_of(int i) const {
        return E % R == 0 || other + i * R < KT ? other + i * R : KT - 1;
    }
    // Where pass i reads its unit (VEC), or place j of it.  koff: byte offsets
    // of the step's k values
    __host__ __device__ __forceinline__ const char* from(const int64_t* koff, int i, int j) const {
        return KW ? at[i] + koff[place[j]] : at[VEC ? 0 : j] + koff[k_of(i)];
    }
    __device__ __forceinline__ void load(const int64_t* koff) {
        constexpr int places = VEC ? 1 : U;
#pragma unroll
        for (int n = 0; n < places * N; ++n) {
            const int i = KW ? n % N : n / places, j = KW ? n / N : n % places;   // one k after the other
            if constexpr (VEC) v[i] = reinterpret_cast<const Loose*>(from(koff, i, 0))->v;
            else v[i][j] = *reinterpret_cast<const T*>(from(koff, i, j));
        }
    }
    // Zeros the k values that do not exist (gone[k] != 0).
    __device__ __forceinline__ void zero(const uint8_t* gone) {
#pragma unroll
        for (int i = 0; i < N; ++i)
#pragma unroll
            for (int j = 0; j < U; ++j)
                if (gone[KW ? place[j] : k_of(i)]) v[i][j] = T(0);
    }
    // whole: the unit's rows are consecutive in LDS
    __device__ __forceinline__ void store(T* lds, bool whole) const {
        if constexpr (!KW && VEC) {
            if (whole) {
#pragma unroll
                for (int i = 0; i < N; ++i)
                    if (live(i)) *reinterpret_cast<Vec*>(lds + L::at(other + i * R, place[0])) = v[i];
                return;
            }
        }
#pragma unroll
        for (int i = 0; i < N; ++i) {
            if (!live(i)) continue;
#pragma unroll
            for (int j = 0; j < U; ++j)
                lds[KW ? L::at(place[j], other + i * R) : L::at(other + i * R, place[j])] = v[i][j];
        }
    }
};

// Byte offsets of a tile's rows in an operand (of a missing row: 0) and in C
// (-1), by ROWS threads from thread `t0` on.
template <typename T, int ROWS>
__device__ __forceinline__ void contract_rows(const ContractGroup& g, int64_t first, int used, int t0, int64_t* o0,
                                              int64_t* o1) {
    const int r = int(threadIdx.x) - t0;
    if (r >= 0 && r < ROWS) {
        int64_t x, y;
        const bool ok = r < used && g.offsets(first + r, &x, &y);
        if (o0) o0[r] = ok ? x * int64_t(sizeof(T)) : 0;
        o1[r] = ok ? y * int64_t(sizeof(T)) : -1;
    }
}

// A lane's part of C: MB x NB blocks, of each four rows of one column (VEC,
// 16-byte accesses) or four columns of one row.  Rows and columns that do not
// exist are read at element 0 and not written.
template <typename T, int MB, int NB, bool VEC>
struct ContractOut {
    using Acc = typename Mma<T>::Acc;
    static constexpr int G = VEC ? 1 : 4;   // column offsets per block
    char* c0;
    int64_t ro[MB], co[NB][G];
    Acc old[MB][NB];

    __device__ __forceinline__ static int row(int lane) { return VEC ? 4 * (lane >> 4) : (lane & 15); }
    __device__ __forceinline__ static int col(int lane) { return VEC ? (lane & 15) : 4 * (lane >> 4); }
    // rows: offsets of the wave's rows, cols: of the tile's columns
    __device__ __forceinline__ void init(T* c, const int64_t* rows, const int64_t* cols) {
        const int lane = threadIdx.x & 63;
        c0 = reinterpret_cast<char*>(c);
#pragma unroll
        for (int i = 0; i < MB; ++i) ro[i] = rows[row(lane) + 16 * i];
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int g = 0; g < G; ++g) co[j][g] = cols[16 * j + col(lane) + g];
    }
    __device__ __forceinline__ void load() {
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const char* c = c0 + (co[j][g] < 0 ? 0 : co[j][g]);
#pragma unroll
                for (int i = 0; i < MB; ++i) {
                    const T* p = reinterpret_cast<const T*>(c + (ro[i] < 0 ? 0 : ro[i]));
                    if constexpr (VEC) old[i][j] = load_rows<T>(p);
                    else old[i][j][g] = *p;
                }
            }
    }
    // alpha * sum, and with UPDATE + beta * what load() read
    template <bool UPDATE>
    __device__ __forceinline__ void store(const Acc (&acc)[MB][NB], T alpha, T beta) const {
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int i = 0; i < MB; ++i) {
                    T* p = reinterpret_cast<T*>(c0 + ro[i] + co[j][g]);
                    const bool ok = ro[i] >= 0 && co[j][g] >= 0;
                    if constexpr (VEC) {
                        Acc out = alpha * acc[i][j];
                        if constexpr (UPDATE) {
                            const Acc pb = beta * old[i][j];
                            out = out + pb;
                        }
                        if (ok) store_rows<T>(p, out);
                    } else {
                        T out = alpha * acc[i][j][g];
                        if constexpr (UPDATE) {
                            const T pb = beta * old[i][j][g];
                            out = out + pb;
                        }
                        if (ok) *p = out;
                    }
                }
    }
};

// Grid: tiles_m * tiles_n * splits workgroups, those from a.first on where
// they take more than one launch.  With one split the tile is
// written to C with alpha and beta; otherwise each split writes its partial
// sums to part[((split * tiles + tile) * NT + column) * MT + row].
//
// A step's operands are loaded into registers over one step and written to LDS
// in the middle of the next (two buffers, one barrier a step), so that neither
// the loads nor the writes are waited for at the barrier.  The offsets of the
// k values are computed for 256 / KT steps at a time, one by each thread.
// VEC: X, Y and C move in whole 16-byte units.
template <typename T, int MB, int NB, bool XK, bool YK, bool VEC>
__global__ __launch_bounds__(256) void k_contract(ContractArgs a, const T* __restrict__ X, const T* __restrict__ Y,
                                                  T* __restrict__ C, T* __restrict__ part, T alpha, T beta,
                                                  int beta0) {
    constexpr int MT = 64 * MB, NT = 16 * NB, KT = contract_kt(sizeof(T), MB);
    using LX = ContractLds<MT, contract_pad(sizeof(T), KT)>;
    using LY = ContractLds<NT, contract_pad(sizeof(T), KT)>;
    using Acc = typename Mma<T>::Acc;
    __shared__ __align__(16) T xs[2][LX::elems(KT)];
    __shared__ __align__(16) T ys[2][LY::elems(KT)];
    __shared__ int64_t row_x[MT], row_c[MT], col_y[NT], col_c[NT];
    // byte offsets of two groups of 256 k values, 0 for those that do not exist
    __shared__ int64_t kx[512], ky[512];
    __shared__ uint8_t gone[512];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t id = a.first + swizzle_id(blockIdx.x, gridDim.x);
    const uint32_t split = a.dv_tiles.div(id), tile = id - split * a.dv_tiles.d;
    const uint32_t tn = a.dv_m.div(tile), tm = tile - tn * a.dv_m.d;
    const int64_t s0 = int64_t(split) * a.split_steps;
    const int steps = int((s0 + a.split_steps < a.steps ? s0 + a.split_steps : a.steps) - s0);

    // k values 256 g .. of the split, g = 0, 1, ...; their entries are kx[(256 g + i) & 511]
    auto k_table = [&](int g) {
        const int i = 256 * g + tid;
        int64_t x, y;
        const bool ok = i < steps * KT && a.k.offsets(s0 * KT + i, &x, &y);
        kx[i & 511] = ok ? x * int64_t(sizeof(T)) : 0;
        ky[i & 511] = ok ? y * int64_t(sizeof(T)) : 0;
        gone[i & 511] = !ok;
    };
    contract_rows<T, MT>(a.m, int64_t(tm) * a.rows, a.rows, 0, row_x, row_c);
    contract_rows<T, NT>(a.n, int64_t(tn) * NT, NT, 256 - NT, col_y, col_c);
    k_table(0);
    __syncthreads();
    ContractLoad<T, MT, KT, XK, VEC> lx;
    ContractLoad<T, NT, KT, YK, VEC> ly;
    const bool whole_x = a.walk_x == 1;
    lx.init(tid, X, row_x, XK ? 1 : a.walk_x, a.walk_y, a.rows);
    ly.init(tid, Y, col_y, XK && YK && a.kwalk_x > 1 ? a.kwalk_y : 1, a.kwalk_x, KT);
    if (steps > 0) {
        lx.load(kx);
        ly.load(ky);
    }
    Acc acc[MB][NB];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[i][j] = Acc{T(0), T(0), T(0), T(0)};
    // VEC: the lane's rows are 4*(lane/16) .. + 3 of column lane % 16 (X's
    // block first); else row lane % 16 of four columns (Y's block first), so
    // that lanes run along C's rows either way
    const int xr = wave * 16 * MB + (VEC ? Mma<T>::frag(lane & 15) : (lane & 15));
    const int yr = VEC ? (lane & 15) : Mma<T>::frag(lane & 15);
    // Only a split's last steps hold k values that do not exist, but for cut
    // labels that do not fill their last chunk.
    const bool holes = XK && YK && a.kwalk_x * a.kwalk_y > 1;
    auto zero = [&](int s) {
        lx.zero(gone + (s * KT & 511));
        ly.zero(gone + (s * KT & 511));
    };
    if (steps > 0) {
        if (holes || steps == 1) zero(0);
        lx.store(xs[0], whole_x);
        ly.store(ys[0], true);
        if (steps > 1) {
            lx.load(kx + KT);
            ly.load(ky + KT);
        }
    }
    __syncthreads();
    // Step s out of buffer b.  Its store writes the next step's tile to LDS
    // half a step before its barrier, its load begins the one after (main:
    // both, unconditionally).
    auto step = [&](int s, auto buffer, auto main) {
        constexpr int Q = KT / 4, b = buffer.value;
        const T* fx0 = xs[b] + (lane >> 4) * LX::LD + xr;
        const T* fy0 = ys[b] + (lane >> 4) * LY::LD + yr;
        T fx[2][MB], fy[2][NB];   // operands are read one product ahead
        auto read = [&](int q) {
#pragma unroll
            for (int i = 0; i < MB; ++i) fx[q & 1][i] = fx0[q * LX::LQ + 16 * i];
#pragma unroll
            for (int j = 0; j < NB; ++j) fy[q & 1][j] = fy0[q * LY::LQ + 16 * j];
        };
        read(0);
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            if (q + 1 < Q) read(q + 1);
            __builtin_amdgcn_sched_barrier(0);   // the reads stay ahead of the products
#pragma unroll
            for (int i = 0; i < MB; ++i)
#pragma unroll
                for (int j = 0; j < NB; ++j)
                    acc[i][j] = VEC ? Mma<T>::step(fx[q & 1][i], fy[q & 1][j], acc[i][j])
                                    : Mma<T>::step(fy[q & 1][j], fx[q & 1][i], acc[i][j]);
            __builtin_amdgcn_sched_barrier(0);
            if (q == Q / 2 - 1 && (main || s + 1 < steps)) {
                if (holes || (!main && s + 2 == steps)) zero(s + 1);
                lx.store(xs[b ^ 1], whole_x);
                ly.store(ys[b ^ 1], true);
                if (main || s + 2 < steps) {
                    lx.load(kx + ((s + 2) * KT & 511));
                    ly.load(ky + ((s + 2) * KT & 511));
                }
            }
        }
        // the group of k values after this step's, into the half that held the
        // one before: the last of those was read three steps ago
        if (s % (256 / KT) == 0) k_table(s / (256 / KT) + 1);
        __syncthreads();
    };
    using B0 = std::integral_constant<int, 0>;
    using B1 = std::integral_constant<int, 1>;
    int s = 0;
    for (; s + 3 < steps; s += 2) {
        step(s, B0{}, std::true_type{});
        step(s + 1, B1{}, std::true_type{});
    }
    for (; s < steps; s += 2) {
        step(s, B0{}, false);
        if (s + 1 < steps) step(s + 1, B1{}, false);
    }
    using Out = ContractOut<T, MB, NB, VEC>;
    if (part) {
        T* p = part + int64_t(id) * (MT * NT) + Out::col(lane) * MT + wave * 16 * MB + Out::row(lane);
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                if constexpr (VEC) {
                    store_rows<T>(p + 16 * j * MT + 16 * i, acc[i][j]);
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r) p[(16 * j + r) * MT + 16 * i] = acc[i][j][r];
                }
            }
        return;
    }
    // C's loads are all in flight before the first use (up to 64 registers)
    Out to;
    to.init(C, row_c + wave * 16 * MB, col_c);
    if (beta0) {
        to.template store<false>(acc, alpha, beta);
    } else {
        to.load();
        to.template store<true>(acc, alpha, beta);
    }
}

// A lane's part of C in C's own order, for kernels that C's traffic bounds: an
// L1 line that one instruction has asked for stalls the next instruction that
// touches it until it arrives, so every access is made to cover whole lines.
// The tile passes through LDS (column by column, rows contiguous) and is
// walked in units of U elements along C: c_run rows, then the columns but for
// a chunk of c_cut that is not next in C, then that chunk, then further rows.
template <typename T, int MT, int NT, int U>
struct ContractWalk {
    static constexpr int N = MT * NT / (256 * U), LDC = MT + 16 / int(sizeof(T));
    typedef T Vec __attribute__((ext_vector_type(U)));
    struct __attribute__((packed, aligned(sizeof(T)))) Loose {
        Vec v;
    };
    int from[N];   // LDS place, -1: beyond the rows in use
    char* p[N];    // in C, null where C has no such element
    Vec old[N];

    __device__ __forceinline__ void init(const ContractArgs& a, T* c, const int64_t* rows, const int64_t* cols) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const uint32_t e = (threadIdx.x + 256 * i) * U;
            const uint32_t q = a.dv_run.div(e), y = e - q * a.dv_run.d;
            const uint32_t x = q / NT, n = q % NT;
            const uint32_t w = a.dv_cut.div(n), col = w + uint32_t(a.c_cut) * (n - w * a.dv_cut.d);
            const uint32_t row = y + a.dv_run.d * x;
            from[i] = int(row) < a.rows ? int(col * LDC + row) : -1;
            const int64_t ro = rows[min(row, uint32_t(MT - 1))], co = cols[col];
            p[i] = from[i] >= 0 && ro >= 0 && co >= 0 ? reinterpret_cast<char*>(c) + ro + co : nullptr;
        }
    }
    __device__ __forceinline__ void load() {
#pragma unroll
        for (int i = 0; i < N; ++i)
            if (p[i]) old[i] = reinterpret_cast<const Loose*>(p[i])->v;
    }
    template <bool UPDATE>
    __device__ __forceinline__ void store(const T* lds, T alpha, T beta) const {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            if (!p[i]) continue;
            Vec out = alpha * *reinterpret_cast<const Vec*>(lds + from[i]);
            if constexpr (UPDATE) {
                const Vec pb = beta * old[i];
                out = out + pb;
            }
            reinterpret_cast<Loose*>(p[i])->v = out;
        }
    }
};

// The operands of a short sum as whole tiles, tile by tile, KT x rows with the
// rows contiguous and zeros for k values that do not exist (rows that do not
// exist hold copies of row 0): workgroup b of all packs X's tile b, or Y's.
template <typename T, int MT, int NT, int KT, bool XK, bool YK, bool VEC>
__global__ __launch_bounds__(256) void k_contract_pack(ContractArgs a, const T* __restrict__ X,
                                                       const T* __restrict__ Y, T* __restrict__ packed) {
    constexpr int PAD = contract_pad(sizeof(T), KT);
    using LX = ContractLds<MT, PAD>;
    using LY = ContractLds<NT, PAD>;
    __shared__ __align__(16) T lds[LX::elems(KT) > LY::elems(KT) ? LX::elems(KT) : LY::elems(KT)];
    __shared__ int64_t rows[MT > NT ? MT : NT], unused[MT > NT ? MT : NT], koff[KT];
    __shared__ uint8_t gone[KT];
    const int tid = threadIdx.x;
    const int64_t id = int64_t(a.first) + blockIdx.x;
    const bool is_x = id < a.tiles_m;
    const int64_t tile = is_x ? id : id - a.tiles_m;
    if (is_x) contract_rows<T, MT>(a.m, tile * a.rows, a.rows, 0, rows, unused);
    else contract_rows<T, NT>(a.n, tile * NT, NT, 0, rows, unused);
    if (tid >= 256 - KT) {
        const int k = tid - (256 - KT);
        int64_t x, y;
        const bool ok = a.k.offsets(k, &x, &y);
        koff[k] = ok ? (is_x ? x : y) * int64_t(sizeof(T)) : 0;
        gone[k] = !ok;
    }
    __syncthreads();
    if (is_x) {
        ContractLoad<T, MT, KT, XK, VEC> l;
        l.init(tid, X, rows, XK ? 1 : a.walk_x, a.walk_y, a.rows);
        l.load(koff);
        l.zero(gone);
        l.store(lds, a.walk_x == 1);
    } else {
        ContractLoad<T, NT, KT, YK, VEC> l;
        l.init(tid, Y, rows, XK && YK && a.kwalk_x > 1 ? a.kwalk_y : 1, a.kwalk_x, KT);
        l.load(koff);
        l.zero(gone);
        l.store(lds, true);
    }
    __syncthreads();
    T* out = packed + (is_x ? tile * (MT * KT) : a.tiles_m * (MT * KT) + tile * (NT * KT));
    const int n = (is_x ? MT : NT) * KT;
    for (int e = tid; e < n; e += 256) {
        const int k = is_x ? e / MT : e / NT;
        out[e] = lds[is_x ? LX::at(k, e % MT) : LY::at(k, e % NT)];
    }
}

// A packed tile on its way to LDS: 16 bytes a thread and pass.
template <typename T, int ROWS, int KT>
struct ContractPacked {
    static constexpr int U = 16 / int(sizeof(T)), N = (ROWS * KT / U + 255) / 256;
    using L = ContractLds<ROWS, contract_pad(sizeof(T), KT)>;
    typedef T Vec __attribute__((ext_vector_type(U)));
    struct __attribute__((packed, aligned(sizeof(T)))) Loose {
        Vec v;
    };
    Vec v[N];
    __device__ __forceinline__ static int unit(int i) { return (int(threadIdx.x) + 256 * i) * U; }
    __device__ __forceinline__ void load(const T* tile) {
#pragma unroll
        for (int i = 0; i < N; ++i)
            if (ROWS * KT / U % 256 == 0 || unit(i) < ROWS * KT) v[i] = reinterpret_cast<const Loose*>(tile + unit(i))->v;
    }
    __device__ __forceinline__ void store(T* lds) const {
#pragma unroll
        for (int i = 0; i < N; ++i)
            if (ROWS * KT / U % 256 == 0 || unit(i) < ROWS * KT)
                *reinterpret_cast<Vec*>(lds + L::at(unit(i) / ROWS, unit(i) % ROWS)) = v[i];
    }
};

// The products of one short sum's tile out of LDS.
template <typename T, int MB, int NB, int KT, bool ROWS_FIRST>
__device__ __forceinline__ void contract_products(const T* xs, const T* ys, typename Mma<T>::Acc (&acc)[MB][NB]) {
    using LX = ContractLds<64 * MB, contract_pad(sizeof(T), KT)>;
    using LY = ContractLds<16 * NB, contract_pad(sizeof(T), KT)>;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[i][j] = typename Mma<T>::Acc{T(0), T(0), T(0), T(0)};
    const int f = Mma<T>::frag(lane & 15), g = lane & 15;
    const T* fx0 = xs + (lane >> 4) * LX::LD + wave * 16 * MB + (ROWS_FIRST ? f : g);
    const T* fy0 = ys + (lane >> 4) * LY::LD + (ROWS_FIRST ? g : f);
#pragma unroll
    for (int q = 0; q < KT / 4; ++q) {
        T fx[MB], fy[NB];
#pragma unroll
        for (int i = 0; i < MB; ++i) fx[i] = fx0[q * LX::LQ + 16 * i];
#pragma unroll
        for (int j = 0; j < NB; ++j) fy[j] = fy0[q * LY::LQ + 16 * j];
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j)
                acc[i][j] = ROWS_FIRST ? Mma<T>::step(fx[i], fy[j], acc[i][j]) : Mma<T>::step(fy[j], fx[i], acc[i][j]);
    }
}

// A sum of at most KT terms: C's traffic bounds the kernel.  C is read before
// the operands (UPDATE).  VECC: C is walked in its own order, and the
// operands' LDS is used again for the result.  PACKED: X points to packed
// tiles of both operands.
template <typename T, int MB, int NB, int KT, bool XK, bool YK, bool VEC, bool PACKED, bool VECC, bool UPDATE>
__global__ __launch_bounds__(256) void k_contract_short(ContractArgs a, const T* __restrict__ X,
                                                        const T* __restrict__ Y, T* __restrict__ C, T alpha, T beta) {
    constexpr int MT = 64 * MB, NT = 16 * NB;
    using LX = ContractLds<MT, contract_pad(sizeof(T), KT)>;
    using LY = ContractLds<NT, contract_pad(sizeof(T), KT)>;
    using Walk = ContractWalk<T, MT, NT, 16 / int(sizeof(T))>;
    constexpr int kOperands = LX::elems(KT) + LY::elems(KT), kResult = VECC ? NT * Walk::LDC : 0;
    __shared__ __align__(16) T lds[kOperands > kResult ? kOperands : kResult];
    T* const xs = lds;
    T* const ys = lds + LX::elems(KT);
    __shared__ int64_t row_c[MT], col_c[NT];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t tile = a.first + swizzle_id(blockIdx.x, gridDim.x);
    const uint32_t tn = a.dv_m.div(tile), tm = tile - tn * a.dv_m.d;
    typename Mma<T>::Acc acc[MB][NB];
    std::conditional_t<VECC, Walk, ContractOut<T, MB, NB, false>> out;
    auto begin_c = [&] {
        if constexpr (VECC) out.init(a, C, row_c, col_c);
        else out.init(C, row_c + wave * 16 * MB, col_c);
        if constexpr (UPDATE) out.load();
    };
    if constexpr (PACKED) {
        ContractPacked<T, MT, KT> lx;
        ContractPacked<T, NT, KT> ly;
        lx.load(X + int64_t(tm) * (MT * KT));
        ly.load(X + a.tiles_m * (MT * KT) + int64_t(tn) * (NT * KT));
        contract_rows<T, MT>(a.m, int64_t(tm) * a.rows, a.rows, 0, nullptr, row_c);
        contract_rows<T, NT>(a.n, int64_t(tn) * NT, NT, 256 - NT, nullptr, col_c);
        __syncthreads();
        begin_c();
        lx.store(xs);
        ly.store(ys);
    } else {
        __shared__ int64_t row_x[MT], col_y[NT], kx[KT], ky[KT];
        __shared__ uint8_t gone[KT];
        contract_rows<T, MT>(a.m, int64_t(tm) * a.rows, a.rows, 0, row_x, row_c);
        contract_rows<T, NT>(a.n, int64_t(tn) * NT, NT, 256 - NT, col_y, col_c);
        if (tid < KT) {
            int64_t x, y;
            const bool ok = a.k.offsets(tid, &x, &y);
            kx[tid] = ok ? x * int64_t(sizeof(T)) : 0;
            ky[tid] = ok ? y * int64_t(sizeof(T)) : 0;
            gone[tid] = !ok;
        }
        __syncthreads();
        begin_c();
        ContractLoad<T, MT, KT, XK, VEC> lx;
        ContractLoad<T, NT, KT, YK, VEC> ly;
        lx.init(tid, X, row_x, XK ? 1 : a.walk_x, a.walk_y, a.rows);
        ly.init(tid, Y, col_y, XK && YK && a.kwalk_x > 1 ? a.kwalk_y : 1, a.kwalk_x, KT);
        lx.load(kx);
        ly.load(ky);
        lx.zero(gone);
        ly.zero(gone);
        lx.store(xs, a.walk_x == 1);
        ly.store(ys, true);
    }
    __syncthreads();
    contract_products<T, MB, NB, KT, VECC>(xs, ys, acc);
    if constexpr (VECC) {
        __syncthreads();   // every wave has read its operands
        T* r0 = lds + (lane & 15) * Walk::LDC + wave * 16 * MB + 4 * (lane >> 4);
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j)
                *reinterpret_cast<typename Mma<T>::Acc*>(r0 + 16 * j * Walk::LDC + 16 * i) = acc[i][j];
        __syncthreads();
        out.template store<UPDATE>(lds, alpha, beta);
    } else {
        out.template store<UPDATE>(acc, alpha, beta);
    }
}

// Sums the splits' partial sums in split order and writes C.  Workgroup b of
// all: 16 columns (b % NB) of tile b / NB.
template <typename T, int MB, int NB>
__global__ __launch_bounds__(256) void k_contract_sum(ContractArgs a, const T* __restrict__ part, T* __restrict__ C,
                                                      int splits, T alpha, T beta, int beta0) {
    constexpr int MT = 64 * MB, NT = 16 * NB, N = 16 * MT / 256;
    __shared__ int64_t row_c[MT], col_c[16];
    const uint32_t id = a.first + blockIdx.x, tile = id / NB, cb = id % NB;
    const uint32_t tn = a.dv_m.div(tile), tm = tile - tn * a.dv_m.d;
    contract_rows<T, MT>(a.m, int64_t(tm) * a.rows, a.rows, 0, nullptr, row_c);
    contract_rows<T, 16>(a.n, int64_t(tn) * NT + 16 * cb, 16, 240, nullptr, col_c);
    __syncthreads();
    const int64_t stride = int64_t(a.dv_tiles.d) * (MT * NT);
    const T* p = part + int64_t(tile) * (MT * NT) + int64_t(16 * cb) * MT + threadIdx.x;
    T sum[N];
#pragma unroll
    for (int i = 0; i < N; ++i) sum[i] = p[256 * i];
    for (int s = 1; s < splits; ++s) {
#pragma unroll
        for (int i = 0; i < N; ++i) sum[i] += p[s * stride + 256 * i];
    }
    const int64_t ro = row_c[threadIdx.x % MT];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int64_t co = col_c[(threadIdx.x + 256 * i) / MT];
        if (ro < 0 || co < 0) continue;
        T* c = reinterpret_cast<T*>(reinterpret_cast<char*>(C) + ro + co);
        *c = beta0 ? alpha * sum[i] : alpha * sum[i] + beta * *c;
    }
}

template <typename T, int MB, int NB>
hipError_t launch_contract_as(const ContractPlan& p, const T* X, const T* Y, T* C, T* part, T alpha, T beta,
                              hipStream_t stream) {
    const int64_t tiles = p.args.tiles_m * p.args.tiles_n;
    if (tiles <= 0) return hipSuccess;
    if (p.args.tiles_m > int64_t(0x7fffffff) || tiles > int64_t(0x7fffffff) / (p.splits > NB ? p.splits : NB))
        return hipErrorInvalidValue;
    T* out = p.splits > 1 ? part : nullptr;
    const int beta0 = beta == T(0);
    ContractArgs a = p.args;
    // launches of at most kContractGroups workgroups that come to `groups`
    auto each = [&](int64_t groups, auto&& launch) {
        for (int64_t first = 0; first < groups; first += kContractGroups) {
            a.first = uint32_t(first);
            launch(dim3(uint32_t(groups - first < kContractGroups ? groups - first : kContractGroups)));
        }
    };
    const dim3 b{256};
    auto go = [&](auto xk, auto yk, auto vec) {
        each(tiles * p.splits, [&](dim3 g) {
            hipLaunchKernelGGL((k_contract<T, MB, NB, xk.value, yk.value, vec.value>), g, b, 0, stream, a, X, Y, C, out,
                               alpha, beta, beta0);
        });
    };
    auto go_short = [&](auto xk, auto yk, auto vec) {
        if constexpr (contract_has_short(sizeof(T), MB, NB)) {
            constexpr int KT = contract_kt(sizeof(T), MB);
            auto with_c = [&](auto packed, auto vecc, auto update) {
                constexpr bool P = packed.value;
                each(tiles, [&](dim3 g) {
                    hipLaunchKernelGGL((k_contract_short<T, MB, NB, KT, !P && xk.value, !P && yk.value, P || vec.value,
                                                         P, vecc.value, update.value>),
                                       g, b, 0, stream, a, P ? part : X, Y, C, alpha, beta);
                });
            };
            auto with_packed = [&](auto packed) {
                if (p.vec_c && beta0) with_c(packed, std::true_type{}, std::false_type{});
                else if (p.vec_c) with_c(packed, std::true_type{}, std::true_type{});
                else if (beta0) with_c(packed, std::false_type{}, std::false_type{});
                else with_c(packed, std::false_type{}, std::true_type{});
            };
            if (p.packed) {
                each(a.tiles_m + a.tiles_n, [&](dim3 g) {
                    hipLaunchKernelGGL((k_contract_pack<T, 64 * MB, 16 * NB, KT, xk.value, yk.value, vec.value>), g, b, 0,
                                       stream, a, X, Y, part);
                });
                with_packed(std::true_type{});
            } else {
                with_packed(std::false_type{});
            }
        }
    };
    const bool is_short = contract_has_short(sizeof(T), MB, NB) && a.steps == 1;
    auto with_vec = [&](auto xk, auto yk) {
        if (is_short && p.vec_xy) go_short(xk, yk, std::true_type{});
        else if (is_short) go_short(xk, yk, std::false_type{});
        else if (p.vec_xy && p.vec_c) go(xk, yk, std::true_type{});
        else go(xk, yk, std::false_type{});
    };
    if (p.xk && p.yk) with_vec(std::true_type{}, std::true_type{});
    else if (p.xk) with_vec(std::true_type{}, std::false_type{});
    else if (p.yk) with_vec(std::false_type{}, std::true_type{});
    else with_vec(std::false_type{}, std::false_type{});
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || p.splits == 1) return e;
    each(tiles * NB, [&](dim3 g) {
        hipLaunchKernelGGL((k_contract_sum<T, MB, NB>), g, b, 0, stream, a, part, C, p.splits, alpha, beta, beta0);
    });
    return hipGetLastError();
}

template <typename T>
hipError_t launch_contract_variant(const ContractPlan& p, const T* X, const T* Y, T* C, T* part, T alpha, T beta,
                                   hipStream_t stream) {
    switch (p.variant) {
#define TTX_CASE(i, mb, nb) \
    case i: return launch_contract_as<T, mb, nb>(p, X, Y, C, part, alpha, beta, stream);
        TTX_CONTRACT_MENU(TTX_CASE)
#undef TTX_CASE
        default: return hipErrorInvalidValue;
    }
}

}  // namespace ttx
