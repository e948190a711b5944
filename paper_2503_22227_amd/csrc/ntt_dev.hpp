// Device code of the negacyclic NTT shared by the single-operation kernels
// (ntt.hip) and the persistent batched kernels (batch.hip).
// Negacyclic NTT / INTT for gfx950 (the paper's butterfly-method NTT, III-A).
//
// Convention: forward output index k holds a(psi^(2 brv(k) + 1)).  The forward
// transform is the radix-2 Cooley-Tukey recursion with psi merged into the
// twiddles: stage st (0-based) pairs j and j + N/2^(st+1) with twiddle
// psi^brv(2^st + j / (N/2^st)).  The inverse runs Gentleman-Sande butterflies
// with psi^-brv(.) from the smallest distance up and folds N^-1 into its last
// stage.
//
// Decomposition: a limb of N = 2^(A+B) residues is seen as a 2^A x 2^B matrix
// (row p, column c at index p 2^B + c).  The first A forward stages only mix
// elements of one column; the last B only mix elements of one row.  So the
// forward transform is a column pass then a row pass, the inverse a row pass
// then a column pass, each a size-2^A or 2^B sub-transform that lives in LDS:
//   * a workgroup owns a 4096-residue tile (32 KiB + padding): 16 columns x
//     256 rows, or 16 rows x 256, so every global access of a wavefront is a
//     run of whole 128-byte lines;
//   * inside the tile every thread holds kElems = 16 residues in registers and
//     performs up to 4 butterfly stages on them (a radix-16 round), then the
//     tile is exchanged through LDS for the next round, so a pass of up to 8
//     stages takes two rounds (256-thread workgroups; 8 residues per thread
//     with radix-8 rounds was measured no faster on MI355X);
//   * primes below 2^46 are transformed in FP64 (ArFp), the others in 64-bit
//     integers that stay in Harvey's lazy ranges ([0, 4q) forward, [0, 2q)
//     inverse) between stages and passes; both are reduced to [0, q) at the
//     last store.
// N <= 4096 is done in one pass by one workgroup per limb.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "modarith.hpp"
#include "rf_internal.hpp"

namespace rf {

constexpr int kTile = 4096;
constexpr int kElems = 16;                         // residues per thread
constexpr int kElemsLog = 4;                       // stages per round
constexpr int kThreads = kTile / kElems;           // threads per workgroup

// Twiddle layout of the row passes.  A row pass of N = 2^(A+B) works on 2^A rows
// of S = 2^B residues, a tile of U = 4096 / S consecutive rows per workgroup,
// T = S / kElems threads per row.  At local stage s (0..B-1) row r uses the
// twiddles j < 2^s of psi^(+-brv(2^(A+s) + r 2^s + j)).  In the round whose
// butterflies only depend on e (the first forward round, the last inverse
// round) j is the same for the T threads of a row; in the other round thread t
// of a row uses j = t R + k, k < R = kElems 2^s / S.  The row table stores them
// so that one wave instruction (consecutive rows u of a tile, then threads t)
// reads consecutive entries:
//   uniform stage: 2^(A+s) + (r_hi 2^s + j) U + u
//   ranged stage:  2^(A+s) + ((r_hi R + k) T + t) U + u,   r = r_hi U + u.
// The entries below 2^A are unused.  A ranged stage is, forward: s >= kElemsLog
// (the stages after the first round); inverse: s >= B - kElemsLog (the stages
// of the first round).
__host__ __device__ constexpr bool row_tw_ranged(int B, bool fwd, int s) {
    return fwd ? s >= kElemsLog : s >= B - kElemsLog;
}

__host__ __device__ inline uint32_t row_tw_index(int A, int B, bool fwd, uint32_t r, int s, uint32_t j) {
    const uint32_t U = (uint32_t)kTile >> B, T = (1u << B) / kElems;
    const uint32_t r_hi = r / U, u = r % U;
    if (!row_tw_ranged(B, fwd, s)) return (1u << (A + s)) + ((r_hi << s) + j) * U + u;
    const uint32_t R = ((uint32_t)kElems << s) >> B;
    const uint32_t t = j / R, k = j % R;
    return (1u << (A + s)) + ((r_hi * R + k) * T + t) * U + u;
}

// Arithmetic of a transform: the register form V of a residue, the twiddles Tw
// and the butterflies.  Between the passes of one transform a residue is kept
// as bits(V) (raw inverts it).
//
// ArInt: 64-bit integers, butterflies with a twiddle w and its 2^62-scaled
// companion wp (shoup62_lazy), nq = 2^64 - q, in Harvey's ranges: inputs and
// outputs below 4q (forward) or 2q (inverse).
struct ArInt {
    using V = uint64_t;
    using Tw = TwPair;
    static constexpr bool kFp = false;
    uint64_t q, q2, nq, ninv, ninv_p, wlast, wlast_p;
    __device__ __forceinline__ explicit ArInt(const PrimeConst &pc)
        : q(pc.q), q2(2 * pc.q), nq(0 - pc.q), ninv(pc.ninv), ninv_p(pc.ninv_p), wlast(pc.wlast),
          wlast_p(pc.wlast_p) {}
    __device__ __forceinline__ static uint64_t bits(V x) { return x; }
    __device__ __forceinline__ static V raw(uint64_t b) { return b; }
    __device__ __forceinline__ void ct(V &x, V &y, const TwPair &w) const {
        uint64_t xr = x >= q2 ? x - q2 : x;               // [0, 2q)
        uint64_t t = shoup62_lazy(y, w.w, w.wp, nq);       // [0, 2q); y < 2^62
        x = xr + t;
        y = xr - t + q2;
    }
    __device__ __forceinline__ void gs(V &x, V &y, const TwPair &w) const {
        uint64_t s = x + y;
        s = s >= q2 ? s - q2 : s;
        uint64_t d = x - y + q2;
        x = s;
        y = shoup62_lazy(d, w.w, w.wp, nq);       // [0, 2q)
    }
    __device__ __forceinline__ void gs_last(V &x, V &y) const {
        uint64_t s = x + y;
        uint64_t d = x - y + q2;
        x = shoup_lazy(s, ninv, ninv_p, q);
        y = shoup_lazy(d, wlast, wlast_p, q);
    }
    // the last inverse stage's output as a residue in [0, q)
    __device__ __forceinline__ uint64_t canon_last(V x) const { return csub(x, q); }
};

// ArFp (primes below kFpPrimeBound): whole numbers in doubles (FpMod), 8 FP64
// operations per butterfly against about 30 integer ones.  Forward, x grows by
// at most 0.75q per stage, 12q over both passes of N = 2^16 and 9q at N = 2^12: from
// inputs below 4q (12q at N = 2^12, where a digit's conversion is a sum of products)
// every value stays below 21q < 2^51, the range mul and red take.  An input may
// also be a whole number of any prime's size (a lift, below 2^46): + 12q is below
// 2^51 as well.  Inverse, the sums double per stage; a round of C
// stages ends by reducing the values that were sums in its last two stages (a
// quarter of them, red()), so that every round starts below 1.5q and its
// sums stay below 24q < 2^51.
struct ArFp {
    using V = double;
    using Tw = double;
    static constexpr bool kFp = true;
    FpMod f;
    double ninv, wlast;
    __device__ __forceinline__ explicit ArFp(const PrimeConst &pc) : f{pc.qd, pc.qinv} {
        ninv = f.centre(pc.ninv);
        wlast = f.centre(pc.wlast);
    }
    __device__ __forceinline__ static uint64_t bits(V x) { return (uint64_t)__double_as_longlong(x); }
    __device__ __forceinline__ static V raw(uint64_t b) { return __longlong_as_double((long long)b); }
    __device__ __forceinline__ void ct(V &x, V &y, double w) const {
        const double t = f.mul(y, w);
        y = x - t;
        x = x + t;
    }
    __device__ __forceinline__ void gs(V &x, V &y, double w) const {
        const double d = x - y;
        x = x + y;
        y = f.mul(d, w);
    }
    __device__ __forceinline__ void gs_last(V &x, V &y) const {
        const double d = x - y;
        x = f.mul(x + y, ninv);
        y = f.mul(d, wlast);
    }
    __device__ __forceinline__ V red(V x) const { return f.red(x); }
    __device__ __forceinline__ uint64_t canon_last(V x) const { return f.canon(x); }
};

// Table index of twiddle j of local stage s: the natural index (tw_base << s) + j
// (column passes, ROW_A == 0) or the row-pass layout above, with tw_base = 2^A + r
// and t the thread's index within its row.
template <int S_LOG, int ROW_A, bool FWD>
__device__ __forceinline__ uint32_t row_or_natural(uint32_t tw_base, int s, int t, uint32_t j) {
    if constexpr (ROW_A == 0) {
        return (tw_base << s) + j;
    } else {
        constexpr uint32_t U = (uint32_t)kTile >> S_LOG, T = (1u << S_LOG) / kElems;
        const uint32_t r = tw_base - (1u << ROW_A);
        const uint32_t r_hi = r / U, uu = r % U;
        if (!row_tw_ranged(S_LOG, FWD, s)) return (1u << (ROW_A + s)) + ((r_hi << s) + j) * U + uu;
        const uint32_t R = ((uint32_t)kElems << s) >> S_LOG;
        return (1u << (ROW_A + s)) + ((r_hi * R + (j - (uint32_t)t * R)) * T + (uint32_t)t) * U + uu;
    }
}

constexpr int ilog2(int x) { return x <= 1 ? 0 : 1 + ilog2(x >> 1); }

// Where a round takes its twiddles: loads from the table as each stage needs
// them (kTwLoad); kTwPrefetch only loads the pairs every round of the pass will
// use into a register array (no butterflies, no LDS access), so that all of
// them are in flight together with the tile's own loads; kTwCached then takes
// them from that array.  A pass with few residues per thread (the small-tile
// passes) otherwise waits one table latency after every round's barrier.
// kTwPrefetchOrdered issues them in the order of the rounds (integer row passes):
// left to the scheduler, a first round waited for the last one's twiddles behind its
// own (2 limbs at N = 2^16, inverse rows 7.1 us against 6.6).  The column passes'
// few twiddles and the FP64 passes' doubles are better left to it (1 to 5 %).
constexpr int kTwLoad = 0, kTwPrefetch = 1, kTwCached = 2, kTwPrefetchOrdered = 3;
constexpr bool tw_prefetch(int tw) { return tw == kTwPrefetch || tw == kTwPrefetchOrdered; }

// Register slots of the prefetched twiddles of a pass of S_LOG stages with E
// residues per thread: round r, group gi, stage c, element e at
// SLOT0(r) + (gi C + c) 2^C + e, each round taking E C slots.  Slots a round
// does not use are never written or read.
__host__ __device__ constexpr int tw_slots(int S_LOG, int E) { return E * S_LOG; }

// Where element p of a thread's sub-transform lies in LDS.  A workgroup tile:
// p ldu + u for sub-transform u.
struct TileLds {
    uint64_t *l;
    int ldu, u;
    __device__ __forceinline__ uint64_t &operator()(int p) const { return l[p * ldu + u]; }
};
// A whole limb, a word of padding after every 16.
struct LimbLds {
    uint64_t *l;
    __device__ __forceinline__ uint64_t &operator()(int p) const { return l[p + (p >> 4)]; }
};

// One round of C butterfly stages of a size-2^S_LOG sub-transform held in LDS
// (element p of the thread's sub-transform at lds(p), as Ar::bits).  Thread t of
// the sub-transform owns E residues (kElems unless stated): E / 2^C groups of
// 2^C residues spaced by the round's smallest distance 2^DL.
//
// IN_REGS / OUT_REGS: the round takes its residues from regs / leaves them in
// regs (group gi, element e at regs[gi * 2^C + e]) instead of LDS.  TW, SLOT0,
// cache: the twiddle source above.
template <typename Ar, int S_LOG, int ST0, int C, bool FWD, bool SCALE_LAST, int ROW_A, bool IN_REGS = false,
          bool OUT_REGS = false, int E = kElems, int TW = kTwLoad, int SLOT0 = 0, typename Lds>
__device__ __forceinline__ void ntt_round(const Lds &lds, int t, uint32_t tw_base,
                                          const typename Ar::Tw *__restrict__ tw, const Ar &ar,
                                          typename Ar::V *regs = nullptr, typename Ar::Tw *cache = nullptr) {
    using V = typename Ar::V;
    using Tw = typename Ar::Tw;
    constexpr int G = 1 << C;
    constexpr int NG = E / G;
    constexpr int DL = FWD ? (S_LOG - ST0 - C) : ST0;
    constexpr bool RUN = !tw_prefetch(TW);
    // twiddle (slot, table index): fetched, loaded or taken from the cache
    auto twiddle = [&](int slot, uint32_t idx) -> Tw {
        if constexpr (tw_prefetch(TW)) {
            cache[slot] = tw[idx];
            return Tw{};
        } else if constexpr (TW == kTwCached) {
            return cache[slot];
        } else {
            return tw[idx];
        }
    };
#pragma unroll
    for (int gi = 0; gi < NG; ++gi) {
        const int grp = t * NG + gi;
        const int lo = grp & ((1 << DL) - 1);
        const int hi = grp >> DL;
        const int base = (hi << (DL + C)) + lo;
        V v[G];
        if constexpr (RUN) {
#pragma unroll
            for (int e = 0; e < G; ++e) {
                if constexpr (IN_REGS) v[e] = regs[gi * G + e];
                else v[e] = Ar::raw(lds(base + (e << DL)));
            }
        }
        if constexpr (FWD) {
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const int st = ST0 + c;
                const int h = G >> (c + 1);
#pragma unroll
                for (int e = 0; e < G; ++e) {
                    if (e & h) continue;
                    // in the first round every group starts below 2^DL, so the twiddle
                    // index depends on e only (uniform across the sub-transform)
                    const uint32_t j = ST0 == 0 ? (uint32_t)(e >> (C - c))
                                                : (uint32_t)((base + (e << DL)) >> (S_LOG - st));
                    const Tw w = twiddle(SLOT0 + (gi * C + c) * G + e,
                                         row_or_natural<S_LOG, ROW_A, true>(tw_base, st, t, j));
                    if constexpr (RUN) ar.ct(v[e], v[e + h], w);
                }
            }
        } else {
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const int us = ST0 + c;
                const int h = 1 << c;
#pragma unroll
                for (int e = 0; e < G; ++e) {
                    if (e & h) continue;
                    if (SCALE_LAST && us == S_LOG - 1) {
                        if constexpr (RUN) ar.gs_last(v[e], v[e + h]);
                    } else {
                        // in the last round every group starts below 2^DL: index from e only
                        const uint32_t lo_part = ST0 + C == S_LOG ? (uint32_t)(e >> (c + 1))
                                                                  : (uint32_t)((base + (e << DL)) >> (us + 1));
                        const Tw w = twiddle(SLOT0 + (gi * C + c) * G + e,
                                             row_or_natural<S_LOG, ROW_A, false>(tw_base, S_LOG - us - 1, t,
                                                                                 lo_part));
                        if constexpr (RUN) ar.gs(v[e], v[e + h], w);
                    }
                }
            }
            // the sums of the round's last two stages (none where it scaled its outputs)
            if constexpr (RUN && Ar::kFp && !(SCALE_LAST && ST0 + C == S_LOG)) {
#pragma unroll
                for (int e = 0; 4 * e < G; ++e) v[e] = ar.red(v[e]);
            }
        }
        if constexpr (RUN) {
#pragma unroll
            for (int e = 0; e < G; ++e) {
                if constexpr (OUT_REGS) regs[gi * G + e] = v[e];
                else lds(base + (e << DL)) = Ar::bits(v[e]);
            }
        }
    }
}

// Rounds of a size-2^S_LOG sub-transform from stage ST0 on: radix-E rounds,
// the last one shorter when log2(E) does not divide S_LOG.  With a prefetch
// only the twiddle loads run (no barriers).
template <typename Ar, int S_LOG, int ST0, bool FWD, bool SCALE_LAST, int ROW_A, int E = kElems, int TW = kTwLoad,
          int SLOT0 = 0, typename Lds>
__device__ __forceinline__ void ntt_rounds_from(const Lds &lds, int t, uint32_t tw_base,
                                                const typename Ar::Tw *__restrict__ tw, const Ar &ar,
                                                typename Ar::Tw *cache = nullptr) {
    constexpr int CL = ilog2(E);
    constexpr int C = (S_LOG - ST0) < CL ? (S_LOG - ST0) : CL;
    constexpr bool LAST = ST0 + C == S_LOG;
    ntt_round<Ar, S_LOG, ST0, C, FWD, SCALE_LAST && LAST, ROW_A, false, false, E, TW, SLOT0>(
        lds, t, tw_base, tw, ar, nullptr, cache);
    if constexpr (!tw_prefetch(TW)) __syncthreads();
    else if constexpr (TW == kTwPrefetchOrdered) __builtin_amdgcn_sched_barrier(0);
    if constexpr (!LAST)
        ntt_rounds_from<Ar, S_LOG, ST0 + C, FWD, SCALE_LAST, ROW_A, E, TW, SLOT0 + E * C>(lds, t, tw_base, tw, ar,
                                                                                         cache);
}

// ROW_A: 0 for the natural twiddle table; A for a row pass reading the row table
// (which needs exactly two rounds of kElems residues: S_LOG in (kElemsLog, 2 kElemsLog]).
template <typename Ar, int S_LOG, bool FWD, bool SCALE_LAST, int ROW_A = 0, int E = kElems, int TW = kTwLoad,
          typename Lds>
__device__ __forceinline__ void ntt_rounds(const Lds &lds, int t, uint32_t tw_base,
                                           const typename Ar::Tw *__restrict__ tw, const Ar &ar,
                                           typename Ar::Tw *cache = nullptr) {
    static_assert(S_LOG >= 5 && S_LOG <= 12, "sub-transform size");
    static_assert(ROW_A == 0 || (E == kElems && S_LOG > kElemsLog && S_LOG <= 2 * kElemsLog),
                  "row table: two rounds of kElems residues");
    ntt_rounds_from<Ar, S_LOG, 0, FWD, SCALE_LAST, ROW_A, E, TW, 0>(lds, t, tw_base, tw, ar, cache);
}

// A prime's twiddles in the form its arithmetic takes.
template <typename Ar>
__device__ __forceinline__ const typename Ar::Tw *twiddles(const TwPair *__restrict__ tw) {
    return reinterpret_cast<const typename Ar::Tw *>(tw);
}

// Blocked layout of a limb between the steps of a key switch or a rescale
// (workspace only, never an operand): blocks of U_r rows x U_c columns, U_r =
// 1024 / 2^B, U_c = 1024 / 2^A, a row of blocks after another.  A tile of 1024
// residues of a row pass is contiguous, as in the natural order, and one of a
// column pass is whole blocks, 128 bytes or more, where the natural order gives
// it 32 bytes a row at N = 2^16: the ModUp column pass of 60 limbs there sends
// the L2s 4.5 million requests against 1.1, at 128 a cycle 16 us of its 28.
// A pass whose both sides are blocked works in place; natural to blocked does not.
constexpr int kBlkLog = 10, kBlkTile = 1 << kBlkLog;

template <int A, int B>
__device__ __forceinline__ size_t blk_index(uint32_t p, uint32_t c) {
    constexpr int LUR = kBlkLog - B, LUC = kBlkLog - A;
    return ((size_t)(p >> LUR) << kBlkLog) + ((c >> LUC) << (LUR + LUC)) + ((p & ((1u << LUR) - 1)) << LUC) +
           (c & ((1u << LUC) - 1));
}

// Memory index of a residue of a column pass.
template <int A, int B, bool BLK>
__device__ __forceinline__ size_t col_index(uint32_t row, uint32_t col) {
    if constexpr (BLK) return blk_index<A, B>(row, col);
    else return ((size_t)row << B) + col;
}

// Row (from the tile's first) and column of the k-th residue in memory of a tile
// of whole rows (at least 1024 residues), BLK: in the blocked layout.
template <int A, int B, bool BLK>
__device__ __forceinline__ void row_elem(int k, int &row, int &col) {
    if constexpr (BLK) {
        constexpr int LUR = kBlkLog - B, LUC = kBlkLog - A;
        const int kk = k & (kBlkTile - 1);
        row = ((k >> kBlkLog) << LUR) + ((kk >> LUC) & ((1 << LUR) - 1));
        col = ((kk >> (LUR + LUC)) << LUC) + (kk & ((1 << LUC) - 1));
    } else {
        row = k >> B;
        col = k & ((1 << B) - 1);
    }
}

// Inputs and outputs of a pass.  A prologue gives the input residue of limb
// index idx, pro(idx) for integer arithmetic and pro.fp(idx, f) (a whole number
// below 2^50 in magnitude) for FP64; an epilogue takes the result, epi(idx, x)
// and epi.fp(idx, x, f).  An element-wise step before or after the transform
// (the ModDown or rescale conversion and tail) runs there instead of in
// another kernel.
template <typename Ar, typename Pro>
__device__ __forceinline__ typename Ar::V pass_in(const Pro &pro, size_t idx, const Ar &ar) {
    if constexpr (Ar::kFp) return pro.fp(idx, ar.f);
    else return pro(idx);
}

template <typename Ar, typename Epi>
__device__ __forceinline__ void pass_out(const Epi &epi, size_t idx, typename Ar::V x, const Ar &ar) {
    if constexpr (Ar::kFp) epi.fp(idx, x, ar.f);
    else epi(idx, x);
}

// Residues in [0, 4q) (no prologue).
struct LoadPro {
    static constexpr bool kBlocked = false;
    const uint64_t *in;
    __device__ __forceinline__ uint64_t operator()(size_t idx) const { return in[idx]; }
    __device__ __forceinline__ double fp(size_t idx, const FpMod &) const { return FpMod::from_u52(in[idx]); }
};

// What the transform's other pass left (the register form's bits); BLK: in the
// blocked layout (row passes).
template <bool BLK>
struct RawInPro {
    static constexpr bool kBlocked = BLK;
    const uint64_t *in;
    __device__ __forceinline__ uint64_t operator()(size_t idx) const { return in[idx]; }
    __device__ __forceinline__ double fp(size_t idx, const FpMod &) const { return ArFp::raw(in[idx]); }
};

using RawPro = RawInPro<false>;
using BlkRawPro = RawInPro<true>;

// Results in [0, q) (the forward transform's last pass).
struct StoreEpi {
    static constexpr bool kPrefetch = false, kBlocked = false;
    uint64_t *out;
    __device__ __forceinline__ void operator()(size_t idx, uint64_t x) const { out[idx] = x; }
    __device__ __forceinline__ void fp(size_t idx, double x, const FpMod &f) const { out[idx] = f.canon(f.red(x)); }
};

// The register form's bits, for the transform's other pass; BLK: in the blocked
// layout (row passes).
template <bool BLK>
struct RawOutEpi {
    static constexpr bool kPrefetch = false, kBlocked = BLK;
    uint64_t *out;
    __device__ __forceinline__ void operator()(size_t idx, uint64_t x) const { out[idx] = x; }
    __device__ __forceinline__ void fp(size_t idx, double x, const FpMod &) const { out[idx] = ArFp::bits(x); }
};

using RawEpi = RawOutEpi<false>;
using BlkRawEpi = RawOutEpi<true>;

// The prologue of a pass and the epilogue of a row pass that are plain loads and stores.
template <bool FIRST>
using PlainPro = std::conditional_t<FIRST, LoadPro, RawPro>;
template <bool FWD, bool BLK>
using RowLoad = std::conditional_t<FWD, RawInPro<BLK>, LoadPro>;
template <bool FWD, bool BLK = false>
using RowStore = std::conditional_t<FWD, StoreEpi, RawOutEpi<BLK>>;

// Tile of a small column pass.  Its U = TILE / 2^A columns are narrower than
// a 128-byte line (G = 16 / U tiles share each line of a row), and workgroups
// are dealt to the 8 XCDs in turn, each with its own L2: dispatch order
// w is mapped so that the G tiles of one line group go to the
// same XCD one after another (w, w + 8, ...), and the line is read from HBM
// once instead of G times.  Identity when the grid is not a multiple of 8 G.
template <int TILE, int A>
__device__ __forceinline__ int xcd_grouped_tile(int w, int tiles) {
    constexpr int U = TILE >> A, G = U >= 16 ? 1 : 16 / U;
    if (G == 1 || tiles % (8 * G) != 0) return w;
    const int x = w & 7, r = w >> 3;
    return ((r / G) * 8 + x) * G + r % G;
}

// Passes of launches with few limbs (the INTT of the special-prime limbs before
// ModDown, the INTT of the dropped limb before a rescale): a tile of TILE
// residues (fewer than kTile) and E residues per thread (fewer than kElems), so
// such a launch has enough workgroups for every CU and a shorter chain of
// dependent butterflies per thread; twiddles from the natural table.  Columns:
// U = TILE / 2^A columns of 2^A rows; rows: U rows of 2^B.  Values in the same
// ranges as the kTile passes (forward columns lazy below 4q, forward rows in
// [0, q); inverse rows lazy below 2q, inverse columns in [0, q)).  Ends with a
// barrier.
template <typename Ar, int A, int B, bool FWD, int TILE, int E, bool BLK = false, typename Pro>
__device__ __forceinline__ void ntt_cols_small_t(uint64_t *lds, const Pro &pro, uint64_t *out,
                                                 const TwPair *__restrict__ tw_all, const Ar &ar, int tile) {
    using V = typename Ar::V;
    constexpr int U = TILE >> A, LDU = U + 1, NT = TILE / E;
    static_assert(U >= 1 && NT >= 64, "small column tile");
    const int col0 = tile * U;
    const auto *tw = twiddles<Ar>(tw_all);
    V vin[E];
#pragma unroll
    for (int r = 0; r < E; ++r) {
        const int idx = threadIdx.x + r * NT;
        vin[r] = pass_in(pro, col_index<A, B, BLK>(idx / U, col0 + idx % U), ar);
    }
    typename Ar::Tw twc[tw_slots(A, E)];
    ntt_rounds<Ar, A, FWD, !FWD, 0, E, kTwPrefetch>(TileLds{lds, LDU, (int)(threadIdx.x % U)}, threadIdx.x / U, 1u, tw, ar, twc);
#pragma unroll
    for (int r = 0; r < E; ++r) {
        const int idx = threadIdx.x + r * NT;
        lds[(idx / U) * LDU + idx % U] = Ar::bits(vin[r]);
    }
    __syncthreads();
    ntt_rounds<Ar, A, FWD, !FWD, 0, E, kTwCached>(TileLds{lds, LDU, (int)(threadIdx.x % U)}, threadIdx.x / U, 1u, tw, ar, twc);
#pragma unroll
    for (int r = 0; r < E; ++r) {
        const int idx = threadIdx.x + r * NT;
        const uint64_t x = lds[(idx / U) * LDU + idx % U];
        out[col_index<A, B, BLK>(idx / U, col0 + idx % U)] = FWD ? x : ar.canon_last(Ar::raw(x));
    }
    __syncthreads();
}

template <int A, int B, bool FWD, int TILE, int E, bool BLK = false, typename Pro>
__device__ __forceinline__ void ntt_cols_small_pro(uint64_t *lds, const Pro &pro, uint64_t *out,
                                                   const TwPair *__restrict__ tw, const PrimeConst &pc, bool fp, int tile) {
    if (fp) ntt_cols_small_t<ArFp, A, B, FWD, TILE, E, BLK>(lds, pro, out, tw, ArFp(pc), tile);
    else ntt_cols_small_t<ArInt, A, B, FWD, TILE, E, BLK>(lds, pro, out, tw, ArInt(pc), tile);
}

template <int A, int B, bool FWD, int TILE, int E, bool BLK>
__device__ __forceinline__ void ntt_cols_small(uint64_t *lds, const uint64_t *in, uint64_t *out,
                                               const TwPair *__restrict__ tw, const PrimeConst &pc, bool fp, int tile) {
    ntt_cols_small_pro<A, B, FWD, TILE, E, BLK>(lds, PlainPro<FWD>{in}, out, tw, pc, fp, tile);
}

// A prologue that computes a thread's residues together (a loop over something
// else outside) takes them all: pro.tile(v, first index, step, ar).
template <typename Pro>
constexpr bool kTilePro = false;

// The result for limb index idx goes through epi (integer: in [0, q) forward,
// lazy in [0, 2q) inverse), or, when Epi::kPrefetch, through
// epi.finish(idx, value, epi.operand(idx)) with the operand loaded at the start.
template <typename Ar, int A, int B, bool FWD, int TILE, int E, typename Pro, typename Epi>
__device__ __forceinline__ void ntt_rows_small_t(uint64_t *lds, const Pro &pro, const TwPair *__restrict__ tw_all,
                                                 const Ar &ar, int tile, const Epi &epi) {
    using V = typename Ar::V;
    constexpr int U = TILE >> B, LDU = U + 1, NT = TILE / E;
    static_assert(U >= 1 && NT >= 64, "small row tile");
    const int row0 = tile * U;
    const auto *tw = twiddles<Ar>(tw_all);
    V vin[E];
    if constexpr (kTilePro<Pro>) {
        pro.tile(vin, ((size_t)row0 << B) + threadIdx.x, NT, ar);
    } else {
#pragma unroll
        for (int r = 0; r < E; ++r) {
            const int idx = threadIdx.x + r * NT;
            vin[r] = pass_in(pro, ((size_t)row0 << B) + idx, ar);
        }
    }
    // an epilogue that reads an operand of its own (the ModDown and rescale
    // tails) has it loaded here, with the tile, instead of after the last
    // barrier: a few registers in a pass of E residues per thread
    uint64_t opnd[E];
    if constexpr (Epi::kPrefetch) {
#pragma unroll
        for (int r = 0; r < E; ++r) {
            const int idx = threadIdx.x + r * NT;
            opnd[r] = epi.operand(((size_t)row0 << B) + idx);
        }
    }
    const int u = threadIdx.x % U;
    typename Ar::Tw twc[tw_slots(B, E)];
    ntt_rounds<Ar, B, FWD, false, 0, E, Ar::kFp ? kTwPrefetch : kTwPrefetchOrdered>(TileLds{lds, LDU, u}, threadIdx.x / U,
                                                                                    (1u << A) + row0 + u, tw, ar, twc);
#pragma unroll
    for (int r = 0; r < E; ++r) {
        const int idx = threadIdx.x + r * NT;
        int row, col;
        row_elem<A, B, Pro::kBlocked>(idx, row, col);
        lds[col * LDU + row] = Ar::bits(vin[r]);
    }
    __syncthreads();
    ntt_rounds<Ar, B, FWD, false, 0, E, kTwCached>(TileLds{lds, LDU, u}, threadIdx.x / U, (1u << A) + row0 + u, tw, ar, twc);
#pragma unroll
    for (int r = 0; r < E; ++r) {
        const int idx = threadIdx.x + r * NT;
        int row, col;
        row_elem<A, B, Epi::kBlocked>(idx, row, col);
        V v = Ar::raw(lds[col * LDU + row]);
        const size_t gi = ((size_t)row0 << B) + idx;
        if constexpr (!Ar::kFp && FWD) v = csub(csub(v, ar.q2), ar.q);
        if constexpr (Epi::kPrefetch) {
            if constexpr (Ar::kFp) epi.finish_fp(gi, v, opnd[r], ar.f);
            else epi.finish(gi, v, opnd[r]);
        } else {
            pass_out(epi, gi, v, ar);
        }
    }
    __syncthreads();
}

template <int A, int B, bool FWD, int TILE, int E, typename Pro, typename Epi>
__device__ __forceinline__ void ntt_rows_small_pe(uint64_t *lds, const Pro &pro, const TwPair *__restrict__ tw,
                                                  const PrimeConst &pc, bool fp, int tile, const Epi &epi) {
    if (fp) ntt_rows_small_t<ArFp, A, B, FWD, TILE, E>(lds, pro, tw, ArFp(pc), tile, epi);
    else ntt_rows_small_t<ArInt, A, B, FWD, TILE, E>(lds, pro, tw, ArInt(pc), tile, epi);
}

template <int A, int B, bool FWD, int TILE, int E, bool BLK>
__device__ __forceinline__ void ntt_rows_small(uint64_t *lds, const uint64_t *in, uint64_t *out,
                                               const TwPair *__restrict__ tw, const PrimeConst &pc, bool fp, int tile) {
    ntt_rows_small_pe<A, B, FWD, TILE, E>(lds, RowLoad<FWD, BLK>{in}, tw, pc, fp, tile, RowStore<FWD, BLK>{out});
}

// Column pass: sub-transforms are columns (2^A rows, stride 2^B), tile
// `tile` covers 4096 / 2^A consecutive columns.  Forward: the first A stages
// (output lazy in [0, 4q)); inverse: the last A stages with the N^-1 scaling
// (output in [0, q)).  The input residue of limb index idx is pro(idx) (a
// plain load, or an element-wise step that precedes the transform: forward
// inputs may lie anywhere in [0, 4q)).
//
// A pass is split into its loads (ntt_cols_load: the kElems input residues of
// this thread, in registers, prologue included) and the rest
// (ntt_cols_compute): the prologue's temporaries are dead before the transform
// starts, which keeps the multi-pass batched kernels within their register
// budget.
// A thread of a 4096-residue tile fetches all its twiddles with its residues
// where they fit the registers: 30 doubles in FP64 (30 pairs of integers, twice
// that, do not).  Fetched stage by stage, each stage waits for the table: the passes of 24
// to 60 limbs at N = 2^16 take 2 to 9 % longer.
template <typename Ar>
__device__ __forceinline__ constexpr int tile_tw() {
    return Ar::kFp ? kTwCached : kTwLoad;
}

template <typename Ar, int A, int B, bool FWD, bool BLK, typename Pro>
__device__ __forceinline__ void ntt_cols_load(typename Ar::V (&regs)[kElems], int tile, const Pro &pro, const Ar &ar) {
    static_assert(A > kElemsLog && A <= 2 * kElemsLog, "two rounds");
    constexpr int U = kTile >> A;
    constexpr int C2 = A - kElemsLog;  // stages of the second round
    const int col0 = tile * U;
    const int u = threadIdx.x % U, t = threadIdx.x / U;
    if constexpr (FWD) {
        // The first forward round works on rows t + e 2^(A-4) of column u, the
        // order in which the tile arrives: it starts from registers.
#pragma unroll
        for (int e = 0; e < kElems; ++e) regs[e] = pass_in(pro, col_index<A, B, BLK>(t + (e << C2), col0 + u), ar);
    } else {
#pragma unroll
        for (int r = 0; r < kTile / kThreads; ++r) {
            const int idx = threadIdx.x + r * kThreads;
            regs[r] = pass_in(pro, col_index<A, B, BLK>(idx / U, col0 + idx % U), ar);
        }
    }
}

// Ends with a barrier, so lds may be reused at once.  The forward output is
// left as Ar's bits (integer: lazy below 4q).
template <typename Ar, int A, int B, bool FWD, bool BLK>
__device__ __forceinline__ void ntt_cols_compute(uint64_t *lds, uint64_t *out, const TwPair *__restrict__ tw_all,
                                                 const Ar &ar, int tile, typename Ar::V (&regs)[kElems],
                                                 typename Ar::Tw *twc) {
    constexpr int S = 1 << A;
    constexpr int U = kTile / S;
    constexpr int LDU = U + 1;
    constexpr int C2 = A - kElemsLog, TW = tile_tw<Ar>(), SLOT1 = kElems * kElemsLog;
    const int col0 = tile * U;
    const int u = threadIdx.x % U, t = threadIdx.x / U;
    const auto *tw = twiddles<Ar>(tw_all);
    if constexpr (FWD) {
        ntt_round<Ar, A, 0, kElemsLog, true, false, 0, true, false, kElems, TW>(TileLds{lds, LDU, u}, t, 1u, tw, ar,
                                                                                regs, twc);
        __syncthreads();
        ntt_round<Ar, A, kElemsLog, C2, true, false, 0, false, false, kElems, TW, SLOT1>(TileLds{lds, LDU, u}, t, 1u,
                                                                                         tw, ar, nullptr, twc);
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kTile / kThreads; ++r) {
            const int idx = threadIdx.x + r * kThreads;
            const int row = idx / U, col = idx % U;
            out[col_index<A, B, BLK>(row, col0 + col)] = lds[row * LDU + col];
        }
    } else {
#pragma unroll
        for (int r = 0; r < kTile / kThreads; ++r) {
            const int idx = threadIdx.x + r * kThreads;
            lds[(idx / U) * LDU + idx % U] = Ar::bits(regs[r]);
        }
        __syncthreads();
        ntt_round<Ar, A, 0, kElemsLog, false, false, 0, false, false, kElems, TW>(TileLds{lds, LDU, u}, t, 1u, tw, ar,
                                                                                  nullptr, twc);
        __syncthreads();
        // The last inverse round leaves rows grp + 16 e (grp = t NG + gi) of
        // column u in registers, the order of a coalesced store.
        ntt_round<Ar, A, kElemsLog, C2, false, true, 0, false, true, kElems, TW, SLOT1>(TileLds{lds, LDU, u}, t, 1u, tw,
                                                                                        ar, regs, twc);
        constexpr int G = 1 << C2, NG = kElems / G;
#pragma unroll
        for (int gi = 0; gi < NG; ++gi)
#pragma unroll
            for (int e = 0; e < G; ++e) {
                const int row = t * NG + gi + (e << kElemsLog);
                out[col_index<A, B, BLK>(row, col0 + u)] = ar.canon_last(regs[gi * G + e]);
            }
    }
    __syncthreads();
}

template <typename Ar, int A, int B, bool FWD, bool BLK = false, typename Pro>
__device__ __forceinline__ void ntt_cols_unit_t(uint64_t *lds, uint64_t *out, const TwPair *__restrict__ tw,
                                                const Ar &ar, int tile, const Pro &pro) {
    typename Ar::V regs[kElems];
    typename Ar::Tw twc[tile_tw<Ar>() == kTwCached ? tw_slots(A, kElems) : 1];
    ntt_cols_load<Ar, A, B, FWD, BLK>(regs, tile, pro, ar);
    if constexpr (tile_tw<Ar>() == kTwCached)
        ntt_rounds<Ar, A, FWD, !FWD, 0, kElems, kTwPrefetch>(TileLds{}, threadIdx.x / (kTile >> A), 1u, twiddles<Ar>(tw),
                                                             ar, twc);
    ntt_cols_compute<Ar, A, B, FWD, BLK>(lds, out, tw, ar, tile, regs, twc);
}

// The prime decides the arithmetic (fp: it is below kFpPrimeBound; uniform
// across the workgroup, a scalar branch).
template <int A, int B, bool FWD, typename Pro>
__device__ __forceinline__ void ntt_cols_unit_pro(uint64_t *lds, uint64_t *out, const TwPair *__restrict__ tw,
                                                  const PrimeConst &pc, bool fp, int tile, const Pro &pro) {
    if (fp) ntt_cols_unit_t<ArFp, A, B, FWD>(lds, out, tw, ArFp(pc), tile, pro);
    else ntt_cols_unit_t<ArInt, A, B, FWD>(lds, out, tw, ArInt(pc), tile, pro);
}

// Launches that hold limbs of both classes give each its own tile: a wide prime's
// is 1024 residues, 4 per thread with every twiddle fetched up front (kMixTile),
// a narrow one's 4096, 16 per thread.  On 4096-residue tiles a wide limb's
// workgroup runs 64 integer butterflies a thread, 3 us of issue and eight waits
// for its twiddles, long after the narrow ones are done: the 13-limb passes at N
// = 2^15 took 9.6 to 15.7 us and take 6.2 to 14.6, the 24 to 60-limb ones at N =
// 2^16 13.4 to 22.0 and now 12.9 to 21.7.
constexpr int kMixTile = 1024, kMixE = kMixTile / kThreads;

template <int A, int B, bool FWD, bool BLK, typename Fp, typename Pro>
__device__ __forceinline__ void ntt_cols_mixed(uint64_t *lds, uint64_t *out, const TwPair *__restrict__ tw,
                                               const PrimeConst &pc, bool fp, int tile, const Pro &pro) {
    if constexpr (std::is_same_v<Fp, WideTiles>) ntt_cols_unit_t<ArInt, A, B, FWD, BLK>(lds, out, tw, ArInt(pc), tile, pro);
    else if (fp) ntt_cols_unit_t<ArFp, A, B, FWD, BLK>(lds, out, tw, ArFp(pc), tile, pro);
    else ntt_cols_small_t<ArInt, A, B, FWD, kMixTile, kMixE, BLK>(lds, pro, out, tw, ArInt(pc), tile);
}

// Rescale / modulus-switch lift as the prologue of the NTT of the lifted limb:
// the last limb x (coefficient domain, in [0, q_l)) taken from its centred
// representative into prime q: [x]_q, + (q - [q_l]_q) when x > q_l / 2, lazy in
// [0, 3q).  KEEP_T (BGV): x is first replaced by [x t^-1]_{q_l} and the result
// multiplied by t (lazy in [0, 2q)), so the lift is 0 mod t as well.  In FP64
// the centred representative of a q_l below kFpPrimeBound is an input as it is.
template <bool KEEP_T>
struct LiftPro {
    static constexpr bool kBlocked = false;
    const uint64_t *last;
    uint64_t ql, ql_half, tinv, tinv_p;  // dropped prime q_l, t^-1 mod q_l
    double qld;                          // q_l in FP64
    uint64_t q, one_p, corr, tmod, tmod_p;
    __device__ __forceinline__ uint64_t lift(uint64_t x) const {
        if (KEEP_T) x = shoup(x, tinv, tinv_p, ql);
        uint64_t r = x - mulhi64(x, one_p) * q;
        if (x > ql_half) r += corr;
        if (KEEP_T) r = shoup_lazy(r, tmod, tmod_p, q);
        return r;
    }
    __device__ __forceinline__ double lift_fp(uint64_t x) const {
        if (KEEP_T || ql >= kFpPrimeBound) return FpMod::from_u52(lift(x));
        const double d = FpMod::from_u52(x);
        return x > ql_half ? d - qld : d;
    }
    __device__ __forceinline__ uint64_t operator()(size_t idx) const { return lift(last[idx]); }
    __device__ __forceinline__ double fp(size_t idx, const FpMod &) const { return lift_fp(last[idx]); }
};

// ModDown base conversion P -> q_i as the prologue of the NTT of target i:
// the K P-limbs y_a (coefficient domain, already multiplied by the input
// factor [(P/p_a)^-1]_{p_a}) give sum_a y_a [P/p_a]_{q_i} + cnt (q_i - [P]_{q_i})
// with cnt the number of y_a above p_a / 2 (centred digits), lazy in [0, 4q).
// KP: the number of special primes K, or 8 for any K <= 8 (runtime K).
template <int KP>
struct ModdownPro {
    static constexpr bool kBlocked = false;
    const uint64_t *src;  // P-limb 0 of the polynomial; limb a at src + a * stride
    size_t stride;
    uint32_t K;
    uint64_t half[KP], cross[KP];
    uint64_t negp, q, r64, r64_p, one_p;
    __device__ __forceinline__ uint64_t operator()(size_t idx) const {
        MacAcc acc;
        uint64_t cnt = 0;
#pragma unroll
        for (int a = 0; a < KP; ++a) {
            if (KP < 8 || a < (int)K) {
                const uint64_t y = src[a * stride + idx];
                cnt += y > half[a] ? 1u : 0u;
                acc.mac(y, cross[a]);
            }
        }
        acc.add(cnt * negp);
        return reduce128_lazy(acc.value(), q, r64, r64_p, one_p);
    }
    __device__ __forceinline__ double fp(size_t idx, const FpMod &) const { return FpMod::from_u52((*this)(idx)); }
};

// Prologue of the first pass of NTT(conv): the ModDown conversion of target i
// of polynomial c from the K P-limbs of ip[c] ([2][nl + K][N]).
template <int KP, int LOGN>
__device__ __forceinline__ ModdownPro<KP> moddown_pro(const uint64_t *ip, const PrimeConst *__restrict__ pcs,
                                                      const PrimeConst &pc, const uint64_t *__restrict__ cross,
                                                      const uint64_t *__restrict__ negp, uint32_t c, uint32_t i,
                                                      uint32_t nl, uint32_t L, uint32_t K) {
    ModdownPro<KP> pro;
    pro.src = ip + (((size_t)c * (nl + K) + nl) << LOGN);
    pro.stride = (size_t)1 << LOGN;
    pro.K = K;
#pragma unroll
    for (int a = 0; a < KP; ++a) {
        pro.half[a] = a < (int)K ? pcs[L + a].q >> 1 : 0;
        pro.cross[a] = a < (int)K ? cross[(size_t)i * K + a] : 0;
    }
    pro.negp = negp[i];
    pro.q = pc.q;
    pro.r64 = pc.r64;
    pro.r64_p = pc.r64_p;
    pro.one_p = pc.one_p;
    return pro;
}

// Prologue of the first pass of NTT(lift): the lift of polynomial c's last
// limb (last [2][N], dropped prime l = nl - 1) into prime i.
template <bool KEEP_T, int LOGN>
__device__ __forceinline__ LiftPro<KEEP_T> lift_pro(const uint64_t *last, const PrimeConst *__restrict__ pcs,
                                                    const PrimeConst &pc, const uint64_t *__restrict__ tab,
                                                    uint32_t c, uint32_t i, uint32_t nl, uint32_t L) {
    const uint32_t l = nl - 1;
    const PrimeConst pl = pcs[l];
    LiftPro<KEEP_T> pro;
    pro.last = last + ((size_t)c << LOGN);
    pro.ql = pl.q;
    pro.ql_half = pl.q >> 1;
    pro.tinv = pl.tinv;
    pro.tinv_p = pl.tinv_p;
    pro.qld = pl.qd;
    pro.q = pc.q;
    pro.one_p = pc.one_p;
    pro.corr = tab[((size_t)l * L + i) * 3 + 2];
    pro.tmod = pc.tmod;
    pro.tmod_p = pc.tmod_p;
    return pro;
}

// Row pass: sub-transforms are rows (2^B contiguous residues), tile `tile`
// covers 4096 / 2^B consecutive rows.  Forward: the last B stages (output in
// [0, q)); inverse: the first B stages (output lazy in [0, 2q)).  The result
// for limb index idx goes through epi(idx, value).  Split into loads and the
// rest like the column pass.
template <typename Ar, int A, int B, typename Pro>
__device__ __forceinline__ void ntt_rows_load(typename Ar::V (&regs)[kElems], int tile, const Pro &pro, const Ar &ar) {
    constexpr int S = 1 << B;
    constexpr int U = kTile / S;
    const int row0 = tile * U;
#pragma unroll
    for (int r = 0; r < kTile / kThreads; ++r) {
        const int idx = threadIdx.x + r * kThreads;
        regs[r] = pass_in(pro, ((size_t)row0 << B) + idx, ar);
    }
}

// BLK_IN: the tile came in the blocked layout.
template <typename Ar, int A, int B, bool FWD, bool BLK_IN, typename Epi>
__device__ __forceinline__ void ntt_rows_compute(uint64_t *lds, const TwPair *__restrict__ tw_all, const Ar &ar,
                                                 int tile, const Epi &epi, typename Ar::V (&regs)[kElems],
                                                 typename Ar::Tw *twc) {
    constexpr int S = 1 << B;
    constexpr int U = kTile / S;
    constexpr int LDU = U + 1;
    const int row0 = tile * U;
    const auto *tw = twiddles<Ar>(tw_all);
#pragma unroll
    for (int r = 0; r < kTile / kThreads; ++r) {
        const int idx = threadIdx.x + r * kThreads;
        int row, col;
        row_elem<A, B, BLK_IN>(idx, row, col);
        lds[col * LDU + row] = Ar::bits(regs[r]);
    }
    __syncthreads();
    const int u = threadIdx.x % U, t = threadIdx.x / U;
    ntt_rounds<Ar, B, FWD, false, A, kElems, tile_tw<Ar>()>(TileLds{lds, LDU, u}, t, (1u << A) + row0 + u, tw, ar, twc);
#pragma unroll
    for (int r = 0; r < kTile / kThreads; ++r) {
        const int idx = threadIdx.x + r * kThreads;
        int row, col;
        row_elem<A, B, Epi::kBlocked>(idx, row, col);
        typename Ar::V x = Ar::raw(lds[col * LDU + row]);
        if constexpr (!Ar::kFp) {
            if (FWD) x = csub(csub(x, ar.q2), ar.q);
        }
        pass_out(epi, ((size_t)row0 << B) + idx, x, ar);
    }
    __syncthreads();
}

template <typename Ar, int A, int B, bool FWD, typename Pro, typename Epi>
__device__ __forceinline__ void ntt_rows_unit_t(uint64_t *lds, const Pro &pro, const TwPair *__restrict__ tw,
                                                const Ar &ar, int tile, const Epi &epi) {
    typename Ar::V regs[kElems];
    typename Ar::Tw twc[tile_tw<Ar>() == kTwCached ? tw_slots(B, kElems) : 1];
    ntt_rows_load<Ar, A, B>(regs, tile, pro, ar);
    if constexpr (tile_tw<Ar>() == kTwCached) {
        constexpr int U = kTile >> B;
        ntt_rounds<Ar, B, FWD, false, A, kElems, kTwPrefetch>(TileLds{}, threadIdx.x / U,
                                                              (1u << A) + tile * U + threadIdx.x % U, twiddles<Ar>(tw),
                                                              ar, twc);
    }
    ntt_rows_compute<Ar, A, B, FWD, Pro::kBlocked>(lds, tw, ar, tile, epi, regs, twc);
}

template <int A, int B, bool FWD, typename Pro, typename Epi>
__device__ __forceinline__ void ntt_rows_unit_pe(uint64_t *lds, const Pro &pro, const TwPair *__restrict__ tw,
                                                 const PrimeConst &pc, bool fp, int tile, const Epi &epi) {
    if (fp) ntt_rows_unit_t<ArFp, A, B, FWD>(lds, pro, tw, ArFp(pc), tile, epi);
    else ntt_rows_unit_t<ArInt, A, B, FWD>(lds, pro, tw, ArInt(pc), tile, epi);
}

// As ntt_cols_mixed; tw_rows: the row-pass layout (4096-residue tiles), tw: the natural one.
template <int A, int B, bool FWD, typename Fp, typename Pro, typename Epi>
__device__ __forceinline__ void ntt_rows_mixed(uint64_t *lds, const Pro &pro, const TwPair *__restrict__ tw_rows,
                                               const TwPair *__restrict__ tw, const PrimeConst &pc, bool fp, int tile,
                                               const Epi &epi) {
    if constexpr (std::is_same_v<Fp, WideTiles>) ntt_rows_unit_t<ArInt, A, B, FWD>(lds, pro, tw_rows, ArInt(pc), tile, epi);
    else if (fp) ntt_rows_unit_t<ArFp, A, B, FWD>(lds, pro, tw_rows, ArFp(pc), tile, epi);
    else ntt_rows_small_t<ArInt, A, B, FWD, kMixTile, kMixE>(lds, pro, tw, ArInt(pc), tile, epi);
}

// The last forward pass with an epilogue of its own, on what the column pass left.
template <int A, int B, typename Epi>
__device__ __forceinline__ void ntt_rows_unit_epi(uint64_t *lds, const uint64_t *in, const TwPair *__restrict__ tw,
                                                  const PrimeConst &pc, bool fp, int tile, const Epi &epi) {
    ntt_rows_unit_pe<A, B, true>(lds, RawPro{in}, tw, pc, fp, tile, epi);
}

// HMult: d2 = a1 b1 mod q as the prologue of the INTT of d2 (the inner product
// computes d0, d1 and its own d2 residues from a and b itself), lazy in
// [0, 2q), the range the inverse butterflies accept.
struct TensorPro {
    static constexpr bool kBlocked = false;
    const uint64_t *a1, *b1;  // limb i of a1, b1
    uint64_t q, r64, r64_p, one_p;
    __device__ __forceinline__ uint64_t operator()(size_t idx) const {
        MacAcc s2;
        s2.mac(a1[idx], b1[idx]);
        return csub(reduce128_lazy(s2.value(), q, r64, r64_p, one_p), 2 * q);
    }
    __device__ __forceinline__ double fp(size_t idx, const FpMod &f) const {
        return f.mul(FpMod::from_u52(a1[idx]), FpMod::from_u52(b1[idx]));
    }
};

// HRotate: sigma_g(a1) as the prologue of its INTT.
struct GatherPro {
    static constexpr bool kBlocked = false;
    const uint64_t *in;  // limb i of a1
    uint32_t galois, log_n;
    __device__ __forceinline__ uint64_t operator()(size_t idx) const {
        return in[galois_src((uint32_t)idx, galois, log_n)];
    }
    __device__ __forceinline__ double fp(size_t idx, const FpMod &) const { return FpMod::from_u52((*this)(idx)); }
};

// ModDown tail as the epilogue of the last forward pass of NTT(conv), the inner
// product having left ip' = ip P^-1 + add: out = ip' - NTT(conv) P^-1 mod q.
struct ModdownFoldEpi {
    // the small-tile row pass loads ip with its tile (operand), then finish
    static constexpr bool kPrefetch = true, kBlocked = false;
    const uint64_t *ip;
    uint64_t *out;
    uint64_t pinv, pinv_p, q;
    __device__ __forceinline__ void operator()(size_t idx, uint64_t conv) const { finish(idx, conv, ip[idx]); }
    __device__ __forceinline__ uint64_t operand(size_t idx) const { return ip[idx]; }
    __device__ __forceinline__ void finish(size_t idx, uint64_t conv, uint64_t ipv) const {
        out[idx] = submod(ipv, shoup(conv, pinv, pinv_p, q), q);
    }
    __device__ __forceinline__ void fp(size_t idx, double conv, const FpMod &f) const { finish_fp(idx, conv, ip[idx], f); }
    __device__ __forceinline__ void finish_fp(size_t idx, double conv, uint64_t ipv, const FpMod &f) const {
        out[idx] = f.canon(f.red(FpMod::from_u52(ipv) - f.mul(conv, f.centre(pinv))));
    }
};

// Rescale / modulus-switch tail as the epilogue of the NTT of the lifted limb:
// out = (in - NTT(lift)) * q_l^-1 mod q.
struct RescaleTailEpi {
    static constexpr bool kPrefetch = true, kBlocked = false;  // as ModdownFoldEpi
    const uint64_t *in;
    uint64_t *out;
    uint64_t qlinv, qlinv_p, q;
    __device__ __forceinline__ void operator()(size_t idx, uint64_t lift) const { finish(idx, lift, in[idx]); }
    __device__ __forceinline__ uint64_t operand(size_t idx) const { return in[idx]; }
    __device__ __forceinline__ void finish(size_t idx, uint64_t lift, uint64_t inv) const {
        out[idx] = shoup(submod(inv, lift, q), qlinv, qlinv_p, q);
    }
    __device__ __forceinline__ void fp(size_t idx, double lift, const FpMod &f) const { finish_fp(idx, lift, in[idx], f); }
    __device__ __forceinline__ void finish_fp(size_t idx, double lift, uint64_t inv, const FpMod &f) const {
        out[idx] = f.canon(f.mul(FpMod::from_u52(inv) - lift, f.centre(qlinv)));
    }
};

// Waves per SIMD the 4096-tile passes are compiled for.  The sub-transforms of
// 2^8 are held to 128 VGPRs, four workgroups per CU: a 60-limb launch at N =
// 2^16 (960 workgroups) is then resident at once.  Measured there, 3 against 4
// waves (130 and 128 VGPRs): forward columns 21.3 against 18.5 us, forward rows
// 22.6 against 19.6 us.  The shorter row transforms would spill 13 to 43
// registers, so they are built for 3.
__host__ __device__ constexpr int ntt_waves(int sub_log) { return sub_log == 8 ? 4 : 3; }
// The lift pass, and the ModDown pass of up to 4 special primes, fit 4 waves at
// every size.
constexpr int kNttWavesFused = 4;

// LDS words a column or row unit needs (the largest tile: 2^8 x 17 padded).
constexpr int kNttLdsWords = 256 * 17;

// Split of log2(N) into the column pass (A stages) and the row pass (B stages).
__host__ __device__ constexpr int ntt_split_a(int log_n) { return (log_n + 1) / 2; }

}  // namespace rf
