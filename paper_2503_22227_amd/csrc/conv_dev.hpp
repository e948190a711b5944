// Device code of the base conversions inside the first pass of the NTT that
// follows them, shared by the single-operation (convert.hip) and the batched
// kernels (batch.hip).
//
// A conversion is a contraction, out_g = sum_k y_k c_{k,g} mod q_g over up to 8
// sources, for every coefficient: on integer units four 30-bit products a term
// and two reductions, 70 instructions an output at 8 sources.  For targets of
// narrow primes the matrix cores take it in bytes: source bytes s_{k,d} (8 a
// source) times the bytes of [2^(8d) c_k]_q taken signed (6 digits), summed over
// the 8 sources x 8 bytes in 32-bit integers, exactly; what is left is one
// combination of six sums, 12 instructions.  A unit takes four targets, so the
// sources are read once for them.  Bound by latency: a workgroup loads, converts,
// transforms and stores once, and all are resident at once or nearly.
// Measured at N = 2^16 with the column pass: ModUp to 60 targets from 8 sources
// 33.1 us in two launches, 23.7 here; ModDown to 48 targets from 4 sources 21.7
// (integer conversion in the 4096-residue pass) and 15.7; N = 2^14, 19 targets
// from 8 sources 11.6 and 7.9.
#pragma once
#include <hip/hip_runtime.h>

#include "ntt_dev.hpp"

namespace rf {

// One wave's tile of 1024 residues of a column pass, 2^A rows of U columns; 16
// rows are followed by a gap, so the second round's rows 16 apart lie on
// different banks.
template <int A>
struct WaveTile {
    static constexpr int U = 1024 >> A, kWords = 1024 + 64 + 16;
    uint64_t *p;
    int u;
    __device__ __forceinline__ static int at(int row, int col) { return row * U + (row >> 4) * U + col; }
    __device__ __forceinline__ uint64_t &operator()(int row) const { return p[at(row, u)]; }
};

typedef int int4v __attribute__((ext_vector_type(4)));

// Sums of products of signed bytes over k: rows of a times columns of b, 16 x 16
// (lane: a's row, b's column lane % 16; bytes (lane / 16) kp / 4 sources; the
// result's column lane % 16, rows 4 (lane / 16) + 0..3).
template <int KP>
__device__ __forceinline__ int4v mac_bytes(const uint64_t (&a)[KP / 4], const uint64_t (&b)[KP / 4]) {
    const int4v zero = {0, 0, 0, 0};
    if constexpr (KP == 8) {
        const int4v x = {(int)(uint32_t)a[0], (int)(a[0] >> 32), (int)(uint32_t)a[1], (int)(a[1] >> 32)};
        const int4v y = {(int)(uint32_t)b[0], (int)(b[0] >> 32), (int)(uint32_t)b[1], (int)(b[1] >> 32)};
        return __builtin_amdgcn_mfma_i32_16x16x64_i8(x, y, zero, 0, 0, 0);
    } else {
        return __builtin_amdgcn_mfma_i32_16x16x32_i8((long)a[0], (long)b[0], zero, 0, 0, 0);
    }
}

// Column pass of up to four narrow targets on tile `tile` (1024 residues) of the
// sources src [s][N].  The four waves convert a quarter of the tile each, for all
// four targets (the matrix instruction's 16 rows: 4 sums of each target, twice),
// then transform a target each, 16 residues a lane.  CENTRED (ModDown): y above
// p / 2 stands for y - p, whose top byte is signed as it is; spc: the sources'
// constants.  frag, off: the block's conversion constants.  Ends with a barrier.
template <int A, int B, int KP, bool CENTRED, bool BLK>
__device__ __forceinline__ void conv_cols_narrow(uint64_t *lds, const uint64_t *src, uint32_t s,
                                                 const PrimeConst *__restrict__ spc, const int8_t *__restrict__ frag,
                                                 const double *__restrict__ off, const TwPair *__restrict__ tw_all,
                                                 const PrimeConst *__restrict__ pcs, const ConvUnit *__restrict__ un,
                                                 uint64_t *dst, int tile) {
    using Tile = WaveTile<A>;
    constexpr int LOGN = A + B, U = Tile::U, NB = KP / 4, H = 8;
    constexpr uint64_t kFlip = 0x0080808080808080ull;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kg = lane >> 4, cg = lane & 15, col0 = tile * U;

    const uint32_t ew = un->e[w];
    const ArFp ar(pcs[ew >> 16]);
    const auto *tw = twiddles<ArFp>(tw_all + ((size_t)(ew >> 16) << LOGN));
    ArFp::Tw twc[tw_slots(A, kElems)];
    const Tile mine{lds + w * Tile::kWords, lane % U};
    ntt_rounds<ArFp, A, true, false, 0, kElems, kTwPrefetch>(mine, lane / U, 1u, tw, ar, twc);

    const int8_t *fr = frag + (size_t)(un->e[cg >> 2] >> 16) * (64 * KP) + ((cg & 3) * KP + kg * NB) * 8;
    uint64_t a0[NB], a1[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        a0[b] = reinterpret_cast<const uint64_t *>(fr)[b];
        a1[b] = reinterpret_cast<const uint64_t *>(fr + 32 * KP)[b];
    }
    const uint32_t gd = un->e[kg] >> 16;
    const double q = pcs[gd].qd, qinv = pcs[gd].qinv, o = off[gd];
    const uint64_t *sp[NB];
    uint64_t p[NB], half[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const uint32_t k = min((uint32_t)(kg * NB + b), s - 1);  // past the sources: times 0
        sp[b] = src + ((size_t)k << LOGN);
        if (CENTRED) {
            p[b] = spc[k].q;
            half[b] = p[b] >> 1;
        }
    }
#pragma unroll
    for (int i0 = 0; i0 < 16; i0 += H) {
        uint64_t y[H][NB];
#pragma unroll
        for (int i = 0; i < H; ++i) {
            const int idx = w * 256 + (i0 + i) * 16 + cg;
#pragma unroll
            for (int b = 0; b < NB; ++b) y[i][b] = sp[b][col_index<A, B, BLK>(idx / U, col0 + idx % U)];
        }
#pragma unroll
        for (int i = 0; i < H; ++i) {
            const int idx = w * 256 + (i0 + i) * 16 + cg;
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                if (CENTRED) y[i][b] -= y[i][b] > half[b] ? p[b] : 0;
                y[i][b] ^= kFlip;
            }
            const int4v d0 = mac_bytes<KP>(a0, y[i]), d1 = mac_bytes<KP>(a1, y[i]);
            // |sums| <= 64 * 2^14: exact below; the top pair 2^32 is reduced first
            const double t0 = d0.x + 256 * d0.y, t1 = d0.z + 256 * d0.w, t2 = d1.x + 256 * d1.y;
            const double h = t2 * 4294967296.0;
            const double c = __builtin_fma(h, qinv, FpMod::kMagic) - FpMod::kMagic;
            const double r = __builtin_fma(-c, q, h) + (__builtin_fma(t1, 65536.0, t0) + o);
            lds[kg * Tile::kWords + Tile::at(idx / U, idx % U)] = ArFp::bits(r);
        }
    }
    __syncthreads();
    ntt_rounds<ArFp, A, true, false, 0, kElems, kTwCached>(mine, lane / U, 1u, tw, ar, twc);
    if (w < (int)un->count) {
        uint64_t *out = dst + ((size_t)(ew & 0xffffu) << LOGN);
#pragma unroll
        for (int r = 0; r < kElems; ++r) {
            const int idx = lane + r * 64;
            out[col_index<A, B, BLK>(idx / U, col0 + idx % U)] = mine.p[Tile::at(idx / U, idx % U)];
        }
    }
    __syncthreads();
}

// ModUp conversion of one target as a prologue: sum_k x_k cross_k, lazy in [0,
// 4q).  A short digit's last source stands in for the missing ones, times 0:
// a branch on each would have the loads wait for one another.
template <int KP>
struct ModupColsPro {
    const uint64_t *src[KP];
    uint64_t cross[KP];
    uint64_t q, r64, r64_p, one_p;
    __device__ __forceinline__ uint64_t operator()(size_t idx) const {
        MacAcc acc;
#pragma unroll
        for (int a = 0; a < KP; ++a)
            acc.mac(src[a][idx], cross[a]);
        return reduce128_lazy(acc.value(), q, r64, r64_p, one_p);
    }
};

// Prologue of target g of a digit of s primes (block blk of the ModUp table).
template <int KP, int LOGN>
__device__ __forceinline__ ModupColsPro<KP> modup_cols_pro(const uint64_t *src, uint32_t s, const uint64_t *cross,
                                                           const PrimeConst &pc) {
    ModupColsPro<KP> pro;
#pragma unroll
    for (int a = 0; a < KP; ++a) {
        pro.src[a] = src + ((size_t)min((uint32_t)a, s - 1) << LOGN);
        pro.cross[a] = a < (int)s ? cross[a] : 0;
    }
    pro.q = pc.q;
    pro.r64 = pc.r64;
    pro.r64_p = pc.r64_p;
    pro.one_p = pc.one_p;
    return pro;
}

// Last pass of a limb's INTT on tile `tile` (1024 residues, blocked layout) by the
// workgroup, its results in [0, q) left in lds at row (U + 1) + column.  Ends with a barrier.
template <typename Ar, int A, int B>
__device__ __forceinline__ void inv_cols_lds(uint64_t *lds, const uint64_t *in, const TwPair *__restrict__ tw_all,
                                             const Ar &ar, int tile) {
    constexpr int U = kMixTile >> A, LDU = U + 1, E = kMixE;
    const auto *tw = twiddles<Ar>(tw_all);
    const TileLds l{lds, LDU, (int)(threadIdx.x % U)};
    uint64_t vin[E];
#pragma unroll
    for (int r = 0; r < E; ++r) {
        const int idx = threadIdx.x + r * kThreads;
        vin[r] = in[blk_index<A, B>(idx / U, tile * U + idx % U)];
    }
    typename Ar::Tw twc[tw_slots(A, E)];
    ntt_rounds<Ar, A, false, true, 0, E, kTwPrefetch>(l, threadIdx.x / U, 1u, tw, ar, twc);
#pragma unroll
    for (int r = 0; r < E; ++r) {
        const int idx = threadIdx.x + r * kThreads;
        lds[(idx / U) * LDU + idx % U] = vin[r];
    }
    __syncthreads();
    ntt_rounds<Ar, A, false, true, 0, E, kTwCached>(l, threadIdx.x / U, 1u, tw, ar, twc);
#pragma unroll
    for (int r = 0; r < E; ++r) {
        const int idx = threadIdx.x + r * kThreads;
        uint64_t &x = lds[(idx / U) * LDU + idx % U];
        x = ar.canon_last(Ar::raw(x));
    }
    __syncthreads();
}

// Column passes of up to four narrow targets of a lift, from inv_cols_lds's tile: a
// wave each, the first round from registers.
template <int A, int B, bool KEEP_T>
__device__ __forceinline__ void lift_cols_narrow(uint64_t *lds, const PrimeConst *__restrict__ pcs,
                                                 const uint64_t *__restrict__ tab, const TwPair *__restrict__ tw_all,
                                                 const ConvUnit *__restrict__ un, uint64_t *dst, uint32_t nl, uint32_t L,
                                                 int tile) {
    using Tile = WaveTile<A>;
    constexpr int LOGN = A + B, U = Tile::U, LDU = U + 1, C2 = A - kElemsLog;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int t = lane / U, u = lane % U;
    const uint32_t i = un->e[w] & 0xffffu;
    const PrimeConst pc = pcs[i];
    const ArFp ar(pc);
    const auto *tw = twiddles<ArFp>(tw_all + ((size_t)i << LOGN));
    const LiftPro<KEEP_T> pro = lift_pro<KEEP_T, LOGN>(nullptr, pcs, pc, tab, 0, i, nl, L);
    ArFp::Tw twc[tw_slots(A, kElems)];
    const Tile mine{lds + w * Tile::kWords, u};
    ntt_rounds<ArFp, A, true, false, 0, kElems, kTwPrefetch>(mine, t, 1u, tw, ar, twc);
    double regs[kElems];
#pragma unroll
    for (int e = 0; e < kElems; ++e) regs[e] = pro.lift_fp(lds[(t + (e << C2)) * LDU + u]);
    __syncthreads();  // the waves' tiles lie over what they have read
    ntt_round<ArFp, A, 0, kElemsLog, true, false, 0, true, false, kElems, kTwCached>(mine, t, 1u, tw, ar, regs, twc);
    __syncthreads();
    ntt_round<ArFp, A, kElemsLog, C2, true, false, 0, false, false, kElems, kTwCached, kElems * kElemsLog>(
        mine, t, 1u, tw, ar, nullptr, twc);
    __syncthreads();
    if (w < (int)un->count) {
        uint64_t *out = dst + ((size_t)i << LOGN);
#pragma unroll
        for (int r = 0; r < kElems; ++r) {
            const int idx = lane + r * 64;
            out[blk_index<A, B>(idx / U, tile * U + idx % U)] = mine.p[Tile::at(idx / U, idx % U)];
        }
    }
}

// The same of one wide target, by the workgroup.
template <int A, int B, bool KEEP_T>
__device__ __forceinline__ void lift_cols_wide(uint64_t *lds, const PrimeConst *__restrict__ pcs,
                                               const uint64_t *__restrict__ tab, const TwPair *__restrict__ tw_all,
                                               uint32_t i, uint64_t *dst, uint32_t nl, uint32_t L, int tile) {
    constexpr int LOGN = A + B, U = kMixTile >> A, LDU = U + 1, E = kMixE;
    const PrimeConst pc = pcs[i];
    const ArInt ar(pc);
    const TwPair *tw = tw_all + ((size_t)i << LOGN);
    const LiftPro<KEEP_T> pro = lift_pro<KEEP_T, LOGN>(nullptr, pcs, pc, tab, 0, i, nl, L);
    const TileLds l{lds, LDU, (int)(threadIdx.x % U)};
    TwPair twc[tw_slots(A, E)];
    ntt_rounds<ArInt, A, true, false, 0, E, kTwPrefetch>(l, threadIdx.x / U, 1u, tw, ar, twc);
#pragma unroll
    for (int r = 0; r < E; ++r) {
        const int idx = threadIdx.x + r * kThreads;
        uint64_t &x = lds[(idx / U) * LDU + idx % U];
        x = pro.lift(x);
    }
    __syncthreads();
    ntt_rounds<ArInt, A, true, false, 0, E, kTwCached>(l, threadIdx.x / U, 1u, tw, ar, twc);
#pragma unroll
    for (int r = 0; r < E; ++r) {
        const int idx = threadIdx.x + r * kThreads;
        dst[((size_t)i << LOGN) + blk_index<A, B>(idx / U, tile * U + idx % U)] = lds[(idx / U) * LDU + idx % U];
    }
}

// LDS of a workgroup: four waves' tiles, or the one tile of a wide target.
template <int A, typename Fp>
constexpr int conv_lds() {
    constexpr int one = (1 << A) * ((kMixTile >> A) + 1), four = 4 * WaveTile<A>::kWords;
    return std::is_same_v<Fp, NoFp> ? one : (four > one ? four : one);
}

}  // namespace rf
