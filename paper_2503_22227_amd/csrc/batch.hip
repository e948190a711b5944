// Batched HMult+Relin over many ciphertexts of different ring degrees and
// levels.  The chain is the single-operation one: INTT of d2 = a1 b1 (formed
// in the first pass), ModUp conversion, NTT, inner product (which forms d0, d1
// and the own-digit d2 residues itself and leaves its Q-limbs as
// ip P^-1 + d_c), INTT of the P-limbs (with the conversion's input factor in
// its last stage), NTT of the ModDown conversion (computed in the first pass,
// the tail out = ip' - NTT(conv) P^-1 in the last).  The tensor,
// ModDown-conversion and tail steps keep their stage numbers with no work
// units.
//
// The ModUp conversion runs in the first pass of its NTT where modup_fused, which
// leaves its own step to the other items.
//
// Launches: each element-wise step (ModUp conversion, inner product) is ONE
// launch over the work units of every item; each NTT pass is one launch per
// ring degree present (one transform shape per kernel keeps the unrolled
// rounds free of register spills).  By default a workgroup takes one work
// unit; rf_batch_set_grid gives a launch a fixed number of workgroups, each
// walking a contiguous range of units (a persistent form the autotuner can
// pick).
//
// Work units: an NTT pass unit is one 4096-residue tile of one limb, or 1024
// residues of a wide limb (kBatchSmallBelow) or of a conversion's targets
// (ConvUnit); an element-wise unit is 256 coefficients of one limb, digit or
// polynomial.  The units of a step are numbered item after
// item (prefix sums in the job tables); a workgroup finds the item of its
// first unit by binary search and then walks forward, so the per-unit
// overhead is a compare.  Mixed ring degrees are dispatched per unit to the
// matching template instantiation of the shared device code (ntt_dev.hpp,
// ks_dev.hpp), so an item's results are bit-identical to the single-operation
// path.  The launch sequence can be captured once in a hipGraph and replayed;
// the job tables are device data, so the graph does not depend on anything but
// the plan.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <vector>

#include "conv_dev.hpp"
#include "ks_dev.hpp"

namespace rf {

// The numbers are rf_batch_set_grid's.  kTensor, kModdownConv and kTail have no
// work units: their work runs inside the passes next to them.
enum BatchStage {
    kTensor = 0,
    kInttD0, kInttD1,       // INTT of d2: row pass, column pass
    kModupConv,
    kNttExt0, kNttExt1,     // NTT of the ModUp output: column pass, row pass
    kInnerProduct,
    kInttP0, kInttP1,       // INTT of the P-limbs
    kModdownConv,
    kNttConv0, kNttConv1,   // NTT of the ModDown conversion
    kTail,
    kStages
};

struct KsJob {
    const uint64_t *a, *b, *evk;
    uint64_t *out;
    uint64_t *d_coeff, *ext, *ip, *conv;
    const PrimeConst *pcs;
    const uint64_t *modup_tab;
    uint64_t modup_stride;
    const uint64_t *pinv;
    uint32_t log_n, nl, L, K, alpha;
    uint32_t unit_begin[kStages];
};

struct NttJob {
    NttBatch b;             // in place but for the first pass of the INTT of d2
    const TwPair *tw_all;   // natural table (column passes, small tiles)
    const TwPair *tw_rows;  // row-pass layout (4096-residue row tiles)
    const PrimeConst *pcs;
    uint32_t log_n;
    uint32_t unit_begin[2];  // first and second pass
    uint32_t small;         // units of the wide limbs, first in b.order, are 1024 residues (limb_units)
    // prologue of the INTT of d2: the item's ciphertexts a, b ([2][nl][N])
    const uint64_t *ct_a, *ct_b;
    // fused conversion before the first pass of NTT(ext), NTT(conv) (conv_dev.hpp; units null: none)
    const ConvUnit *units;
    const int8_t *frag;
    const double *off;
    const uint64_t *x, *modup_tab;  // ModUp: d_coeff, table
    uint64_t modup_stride;
    // ModDown in NTT(conv): conversion from the P-limbs of ip in the first pass,
    // tail out = ip' - NTT(conv) P^-1 in the last
    const uint64_t *ip;
    uint64_t *out;
    const uint64_t *pinv, *md_cross, *md_negp;
    uint32_t nl, K, L, alpha;
};

template <typename J>
__device__ __forceinline__ uint32_t unit_begin_of(const J &j, int stage);
template <>
__device__ __forceinline__ uint32_t unit_begin_of<KsJob>(const KsJob &j, int stage) {
    return j.unit_begin[stage];
}
template <>
__device__ __forceinline__ uint32_t unit_begin_of<NttJob>(const NttJob &j, int pass) {
    return j.unit_begin[pass];
}

// The pointers of a job table address device memory, but loaded from the table
// they are generic pointers, and every access through one would be a flat
// instruction (counted by both the vector-memory and the LDS/scalar wait
// counters, so each use waits for both).  A job is copied with its pointers'
// bits re-typed as global-address-space pointers, which lets the compiler emit
// global loads and stores.
template <typename T>
__device__ __forceinline__ T *gptr(T *p) {
    return (T *)(__attribute__((address_space(1))) T *)(uintptr_t)p;
}

__device__ __forceinline__ KsJob global_job(const KsJob &J) {
    KsJob g = J;
    g.a = gptr(J.a);
    g.b = gptr(J.b);
    g.evk = gptr(J.evk);
    g.out = gptr(J.out);
    g.d_coeff = gptr(J.d_coeff);
    g.ext = gptr(J.ext);
    g.ip = gptr(J.ip);
    g.conv = gptr(J.conv);
    g.pcs = gptr(J.pcs);
    g.modup_tab = gptr(J.modup_tab);
    g.pinv = gptr(J.pinv);
    return g;
}

__device__ __forceinline__ NttJob global_job(const NttJob &J) {
    NttJob g = J;
    g.b.in = gptr(J.b.in);
    g.b.out = gptr(J.b.out);
    g.b.order.ent = gptr(J.b.order.ent);
    g.tw_all = gptr(J.tw_all);
    g.tw_rows = gptr(J.tw_rows);
    g.pcs = gptr(J.pcs);
    g.ct_a = gptr(J.ct_a);
    g.ct_b = gptr(J.ct_b);
    g.ip = gptr(J.ip);
    g.out = gptr(J.out);
    g.pinv = gptr(J.pinv);
    g.md_cross = gptr(J.md_cross);
    g.md_negp = gptr(J.md_negp);
    g.units = gptr(J.units);
    g.frag = gptr(J.frag);
    g.off = gptr(J.off);
    g.x = gptr(J.x);
    g.modup_tab = gptr(J.modup_tab);
    return g;
}

// Last job whose first unit is <= u (jobs sorted by unit_begin).
template <typename J>
__device__ __forceinline__ uint32_t find_job(const J *jobs, uint32_t njobs, uint32_t u, int stage) {
    uint32_t lo = 0, hi = njobs;
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (unit_begin_of(jobs[mid], stage) <= u) lo = mid;
        else hi = mid;
    }
    return lo;
}

// CH: ModUp conversion output limbs per thread (kModupConv only).
template <int STAGE, int CH = kModupChunk>
__global__ __launch_bounds__(kEw) void ks_batched_kernel(const KsJob *__restrict__ jobs, uint32_t njobs,
                                                         uint32_t total, uint32_t per_wg) {
    const uint32_t u0 = blockIdx.x * per_wg;
    const uint32_t u1 = min(total, u0 + per_wg);
    if (u0 >= u1) return;
    uint32_t j = find_job(jobs, njobs, u0, STAGE);
    for (uint32_t u = u0; u < u1; ++u) {
        while (j + 1 < njobs && jobs[j + 1].unit_begin[STAGE] <= u) ++j;
        const KsJob J = global_job(jobs[j]);
        const uint32_t local = u - J.unit_begin[STAGE];
        const uint32_t cshift = J.log_n - 8;  // N / 256 blocks per row
        const uint32_t gy = local >> cshift, gx = local & ((1u << cshift) - 1);
        if constexpr (STAGE == kModupConv) {
            modup_bconv_unit<true, CH>(J.d_coeff, J.ext, J.pcs, J.modup_tab, J.modup_stride, J.log_n, J.nl, J.L, J.K, J.alpha,
                             gx, gy);
        } else {
            IpFold f;
            f.pinv = J.pinv;
            f.mode = 1;
            f.a = J.a;
            f.b = J.b;
            inner_product_unit<1>(nullptr, J.ext, J.evk, J.ip, J.pcs, J.log_n, J.nl, J.L, J.K, J.alpha, gx, gy, f);
        }
    }
}

// The NTT passes of a batch.  The transforms' coefficient sides and what lies
// between their passes are in the blocked layout (ntt_dev.hpp).
enum BatchPass {
    kPassTensor,    // INTT of d2 = a1 b1: rows
    kPassInvRows,   // INTT of the P-limbs: rows
    kPassInvCols,   // either's columns
    kPassModup,     // NTT of the extension: columns, with the conversion where it is fused
    kPassFwdRows,   // its rows
    kPassModdown4,  // NTT of the ModDown conversion: columns and the conversion from 4 special primes
    kPassModdown8,  // or any number up to 8
    kPassTail       // its rows, with the tail
};
__host__ __device__ constexpr bool pass_cols(int p) {
    return p == kPassInvCols || p == kPassModup || p == kPassModdown4 || p == kPassModdown8;
}
__host__ __device__ constexpr int pass_second(int p) {
    return p == kPassInvCols || p == kPassFwdRows || p == kPassTail;
}

// Unit `local` of a job's limbs.
struct BatchUnit {
    uint32_t li, poly, g;
    int tile;
    int kind;  // 0: a wide limb's 4096 residues, 1: its 1024, 2: a narrow one's 4096
};
template <int LOGN>
__device__ __forceinline__ BatchUnit batch_unit(const NttJob &J, uint32_t local) {
    constexpr int TW = LOGN - 10, TN = LOGN - 12;
    BatchUnit u;
    uint32_t e;
    const uint32_t wide = J.b.order.n_wide * J.b.n_polys, tw = J.small ? TW : TN;
    if (local < wide << tw) {
        u.kind = J.small ? 1 : 0;
        e = local >> tw;
        u.tile = local & ((1 << tw) - 1);
    } else {
        u.kind = 2;
        local -= wide << tw;
        e = wide + (local >> TN);
        u.tile = local & ((1 << TN) - 1);
    }
    const uint32_t k = J.b.n_polys == 1 ? e : e >> 1;
    u.poly = J.b.n_polys == 1 ? 0 : e & 1;
    const uint32_t x = J.b.order.ent[k];
    u.li = x & 0xffffu;
    u.g = x >> 16;
    return u;
}

template <int A, int B, bool FWD, typename Fp, typename Pro, typename Epi>
__device__ __forceinline__ void batch_rows(uint64_t *lds, const NttJob &J, const BatchUnit &u, const PrimeConst &pc,
                                           const Pro &pro, const Epi &epi) {
    const size_t t = (size_t)u.g << (A + B);
    if (!std::is_same_v<Fp, NoFp> && u.kind == 2) ntt_rows_unit_t<ArFp, A, B, FWD>(lds, pro, J.tw_rows + t, ArFp(pc), u.tile, epi);
    else if (u.kind == 1) ntt_rows_small_t<ArInt, A, B, FWD, kMixTile, kMixE>(lds, pro, J.tw_all + t, ArInt(pc), u.tile, epi);
    else ntt_rows_unit_t<ArInt, A, B, FWD>(lds, pro, J.tw_rows + t, ArInt(pc), u.tile, epi);
}

// Column pass with a ModUp conversion: unit `local` of the extension's units.
template <int A, int B, int KP, typename Fp>
__device__ __forceinline__ void batch_modup(uint64_t *lds, const NttJob &J, uint32_t local) {
    constexpr int LOGN = A + B, TL = LOGN - 10;
    const int tile = xcd_grouped_tile<kMixTile, A>(local & ((1 << TL) - 1), 1 << TL);
    const ConvUnit *un = J.units + (local >> TL);
    const uint32_t j = un->digit, s = un->size, blk = j * J.alpha + s - 1;
    const uint64_t *src = J.x + ((size_t)j * J.alpha << LOGN);
    uint64_t *dst = J.b.out + ((size_t)j * (J.nl + J.K - J.alpha) << LOGN);
    if (std::is_same_v<Fp, NoFp> || un->wide) {
        const uint32_t li = un->e[0] & 0xffffu, g = un->e[0] >> 16;
        const PrimeConst pc = J.pcs[g];
        const ModupColsPro<KP> pro = modup_cols_pro<KP, LOGN>(
            src, s, J.modup_tab + blk * J.modup_stride + 2 * J.alpha + (size_t)g * J.alpha, pc);
        ntt_cols_small_t<ArInt, A, B, true, kMixTile, kMixE, true>(lds, pro, dst + ((size_t)li << LOGN),
                                                                   J.tw_all + ((size_t)g << LOGN), ArInt(pc), tile);
    } else if constexpr (!std::is_same_v<Fp, NoFp>) {
        const size_t b = (size_t)blk * (J.L + J.K);
        conv_cols_narrow<A, B, KP, false, true>(lds, src, s, nullptr, J.frag + b * (64 * KP), J.off + b, J.tw_all, J.pcs,
                                                un, dst, tile);
    }
}

// One pass over unit u of a job.
template <int A, int B, int PASS, typename Fp>
__device__ __forceinline__ void ntt_batched_unit(uint64_t *lds, const NttJob &J, uint32_t u) {
    constexpr int LOGN = A + B;
    const uint32_t local = u - J.unit_begin[pass_second(PASS)];
    if constexpr (PASS == kPassModup) {
        if (J.units) {
            if (J.alpha <= 4) batch_modup<A, B, 4, Fp>(lds, J, local);
            else batch_modup<A, B, 8, Fp>(lds, J, local);
            return;
        }
    }
    if constexpr (PASS == kPassModdown4 || PASS == kPassModdown8) {
        constexpr int KP = PASS == kPassModdown4 ? 4 : 8;
        if (J.units) {
            constexpr int TL = LOGN - 10;
            const int tile = xcd_grouped_tile<kMixTile, A>(local & ((1 << TL) - 1), 1 << TL);
            const uint32_t w = local >> TL, poly = w & 1;
            const ConvUnit *un = J.units + (w >> 1);
            uint64_t *dst = J.b.out + ((size_t)poly * J.nl << LOGN);
            if (std::is_same_v<Fp, NoFp> || un->wide) {
                const uint32_t i = un->e[0] & 0xffffu;
                const PrimeConst pc = J.pcs[i];
                ntt_cols_small_t<ArInt, A, B, true, kMixTile, kMixE, true>(
                    lds, moddown_pro<KP, LOGN>(J.ip, J.pcs, pc, J.md_cross, J.md_negp, poly, i, J.nl, J.L, J.K),
                    dst + ((size_t)i << LOGN), J.tw_all + ((size_t)i << LOGN), ArInt(pc), tile);
            } else if constexpr (!std::is_same_v<Fp, NoFp>) {
                const uint64_t *src = J.ip + (((size_t)poly * (J.nl + J.K) + J.nl) << LOGN);
                if (KP == 4 || J.K <= 4)
                    conv_cols_narrow<A, B, 4, true, true>(lds, src, J.K, J.pcs + J.L, J.frag, J.off, J.tw_all, J.pcs, un,
                                                          dst, tile);
                else
                    conv_cols_narrow<A, B, 8, true, true>(lds, src, J.K, J.pcs + J.L, J.frag, J.off, J.tw_all, J.pcs, un,
                                                          dst, tile);
            }
            return;
        }
    }
    const BatchUnit w = batch_unit<LOGN>(J, local);
    const PrimeConst pc = J.pcs[w.g];
    const size_t t = (size_t)w.g << LOGN;
    uint64_t *out = J.b.out + (size_t)w.poly * J.b.out_poly_stride + ((size_t)w.li << LOGN);
    if constexpr (PASS == kPassTensor) {
        // d2 = a1 b1 of limb li
        const size_t poly1 = ((size_t)J.nl + w.li) << LOGN;
        const TensorPro pro{J.ct_a + poly1, J.ct_b + poly1, pc.q, pc.r64, pc.r64_p, pc.one_p};
        batch_rows<A, B, false, Fp>(lds, J, w, pc, pro, BlkRawEpi{out});
    } else if constexpr (PASS == kPassInvRows) {
        batch_rows<A, B, false, Fp>(lds, J, w, pc, LoadPro{out}, BlkRawEpi{out});
    } else if constexpr (PASS == kPassFwdRows) {
        batch_rows<A, B, true, Fp>(lds, J, w, pc, BlkRawPro{out}, StoreEpi{out});
    } else if constexpr (PASS == kPassTail) {
        // limb li of polynomial poly of conv [2][nl][N]: ModDown tail into out
        const size_t lo = ((size_t)w.poly * (J.nl + J.K) + w.li) << LOGN;
        const size_t oo = ((size_t)w.poly * J.nl + w.li) << LOGN;
        batch_rows<A, B, true, Fp>(lds, J, w, pc, BlkRawPro{out},
                               ModdownFoldEpi{J.ip + lo, J.out + oo, J.pinv[2 * w.li], J.pinv[2 * w.li + 1], pc.q});
    } else if constexpr (PASS == kPassInvCols) {
        if (!std::is_same_v<Fp, NoFp> && w.kind == 2) ntt_cols_unit_t<ArFp, A, B, false, true>(lds, out, J.tw_all + t, ArFp(pc), w.tile, RawPro{out});
        else if (w.kind == 1)
            ntt_cols_small_t<ArInt, A, B, false, kMixTile, kMixE, true>(lds, RawPro{out}, out, J.tw_all + t, ArInt(pc),
                                                                        xcd_grouped_tile<kMixTile, A>(w.tile, 1 << (LOGN - 10)));
        else ntt_cols_unit_t<ArInt, A, B, false, true>(lds, out, J.tw_all + t, ArInt(pc), w.tile, RawPro{out});
    } else if constexpr (PASS == kPassModup) {
        // wide primes alone, several a digit: converted by a launch of their own
        if (w.kind == 1)
            ntt_cols_small_t<ArInt, A, B, true, kMixTile, kMixE, true>(lds, LoadPro{out}, out, J.tw_all + t, ArInt(pc),
                                                                       xcd_grouped_tile<kMixTile, A>(w.tile, 1 << (LOGN - 10)));
        else ntt_cols_unit_t<ArInt, A, B, true, true>(lds, out, J.tw_all + t, ArInt(pc), w.tile, LoadPro{out});
    } else {
        constexpr int KP = PASS == kPassModdown4 ? 4 : 8;
        ntt_cols_unit_t<ArInt, A, B, true, true>(
            lds, out, J.tw_all + t, ArInt(pc), w.tile,
            moddown_pro<KP, LOGN>(J.ip, J.pcs, pc, J.md_cross, J.md_negp, w.poly, w.li, J.nl, J.L, J.K));
    }
}

// One pass of a batched (I)NTT over the items of one ring degree 2^(A+B) (the
// plan launches each NTT step once per ring degree present: one transform
// shape per kernel keeps the unrolled rounds free of register spills).  Units
// [unit0, unit0 + total) of the step; jobs = the items of the ring degree, whose
// unit_begin values are absolute.  LOOP: workgroups walk per_wg consecutive
// units; otherwise each takes one unit (per_wg == 1).  The loop keeps every
// path's addresses in registers: at 2 waves per SIMD it hardly spills (at 4, 52 to 143
// registers: 64 items of N = 2^14..2^16 with 2048 workgroups a launch 5085 us, and 3858).
template <int A, int B, int PASS, bool LOOP, typename Fp>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(LOOP ? 2 : PASS == kPassModdown8 ? 3 : ntt_waves(pass_cols(PASS) ? A : B)))) void ntt_batched_kernel(
    const NttJob *__restrict__ jobs, uint32_t njobs, uint32_t unit0, uint32_t total, uint32_t per_wg) {
    constexpr bool COLS = pass_cols(PASS);
    constexpr int kTileWords = COLS ? (1 << A) * (kTile / (1 << A) + 1) : (1 << B) * (kTile / (1 << B) + 1);
    constexpr int kConvWords = COLS ? conv_lds<A, Fp>() : 0;
    __shared__ uint64_t lds[kTileWords > kConvWords ? kTileWords : kConvWords];
    constexpr int pass = pass_second(PASS);
    if constexpr (!LOOP) {
        if (blockIdx.x >= total) return;
        const uint32_t u = unit0 + blockIdx.x;
        ntt_batched_unit<A, B, PASS, Fp>(lds, global_job(jobs[find_job(jobs, njobs, u, pass)]), u);
    } else {
        const uint32_t u0 = unit0 + blockIdx.x * per_wg;
        const uint32_t u1 = unit0 + min(total, (blockIdx.x + 1) * per_wg);
        if (u0 >= u1) return;
        uint32_t j = find_job(jobs, njobs, u0, pass);
        for (uint32_t u = u0; u < u1; ++u) {
            while (j + 1 < njobs && jobs[j + 1].unit_begin[pass] <= u) ++j;
            ntt_batched_unit<A, B, PASS, Fp>(lds, global_job(jobs[j]), u);
        }
    }
}

}  // namespace rf

using namespace rf;

struct rf_batch {
    int device = 0;
    uint32_t n_items = 0;
    // items sorted by ring degree; group: [job0, job1) with one log_n, and the
    // first unit / unit count of every step inside the group
    struct Group {
        uint32_t log_n, job0, job1;
        bool k4;  // every item has 4 special primes (the specialised ModDown prologue)
        // no item has a narrow prime: kernels of the integer code alone (a workgroup a
        // unit), 14 limbs of 55 bits at N = 2^15, 8 items 884 and 873 us, 12 of 60 bits at
        // N = 2^16, 8 items 624 and 616
        bool wide;
        uint32_t unit0[kStages], units[kStages];
    };
    std::vector<Group> groups;
    KsJob *d_jobs = nullptr;
    NttJob *d_ntt[4] = {nullptr, nullptr, nullptr, nullptr};  // INTT d2, NTT ext, INTT P, NTT conv
    uint32_t total[kStages] = {0};
    uint32_t grid[kStages] = {0};  // workgroups per launch; 0 = one per unit
    uint32_t modup_chunk = kModupChunk;  // ModUp output limbs per thread
    std::vector<rf_batch_item> items;    // the item list, to rebuild the tables
    uint64_t *ws = nullptr;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    hipStream_t capture_stream = nullptr;
};

namespace {

// (nl of them spare)
size_t item_ws_limbs(const rf_ctx *c, uint32_t nl) {
    const ModupLevel &lv = c->modup_levels[nl];
    return (size_t)nl + (size_t)nl + lv.ext_limbs + 2 * (size_t)(nl + c->K) + 2 * (size_t)nl;
}

int validate(const rf_batch_item *items, uint32_t n) {
    if (!items || n == 0) return fail(RF_EINVAL, "rf_batch: no items");
    const rf_ctx *c0 = items[0].ctx;
    for (uint32_t i = 0; i < n; ++i) {
        const rf_batch_item &it = items[i];
        const rf_ctx *c = it.ctx;
        if (!c || !it.a || !it.b || !it.rlk || !it.out) return fail(RF_EINVAL, "rf_batch: null pointer in an item");
        if (c->scheme != RF_CKKS && c->scheme != RF_BGV) return fail(RF_EUNSUPPORTED, "rf_batch: CKKS or BGV");
        if (c->log_n < 13 || c->log_n > 16) return fail(RF_EUNSUPPORTED, "rf_batch: ring degree 2^13..2^16");
        if (it.n_limbs < 1 || it.n_limbs > c->L) return fail(RF_ELEVEL, "rf_batch: limb count out of range");
        if (c->device != c0->device) return fail(RF_EINVAL, "rf_batch: items on different devices");
        if (it.out == it.a || it.out == it.b) return fail(RF_EINVAL, "rf_batch: out aliases an input");
    }
    return RF_OK;
}

// Job list of an NTT step: INTT of d2, NTT of ext, INTT of the P-limbs, NTT of conv.
int list_of(int st) {
    return st == kInttD0 || st == kInttD1 ? 0 : st == kNttExt0 || st == kNttExt1 ? 1 : st == kInttP0 || st == kInttP1 ? 2 : 3;
}

// The wide limbs of a launch (one job list, one ring degree) go in 1024-residue
// tiles, ahead of the narrow ones', where it holds fewer 4096-residue tiles than two
// a CU: a 4096-residue workgroup of a wide limb runs three times a narrow one's time
// and would end last.  Fuller launches are bound by what all of them issue, of
// which the larger tile takes less.  Row passes in 4096 and in 1024, tiles (wide ones
// among them): P-limbs 64 11.1 and 7.5 us, 256 13.0 and 12.6, 512 18.2 and 20.5, 1024
// 28.6 and 34.1; extension 144 (72) 11.4 and 9.4, 576 (288) 16.9 and 17.8, 1152 (960)
// 27.3 and 32.1, 4608 (3840) 73 and 104; ModDown's 192 (48) 15.5 and 14.2, 768 (192)
// 21.8 and 24.5.  The pass that forms d2 = a1 b1 gains from the smaller ones while they
// are few: 768 (64) 23.6 and 18.7, 1536 (384) 37.5 and 33.5, 1536 (1152) 41.2 and 44.2.
constexpr uint64_t kBatchSmallBelow = 512;
bool batch_small(int list, uint64_t wide, uint64_t tiles) {
    return tiles < kBatchSmallBelow || (list == 0 && wide * 3 <= tiles);
}

// Units of a pass over np polynomials of `limbs` limbs, n_wide of them wide, those
// in tiles of 1024 residues if small (batch_unit), else all in 4096.
uint32_t limb_units(const rf_ctx *c, uint32_t limbs, uint32_t n_wide, uint32_t np, bool small) {
    return np * (n_wide * (c->n / (small ? kMixTile : kTile)) + (limbs - n_wide) * (c->n / kTile));
}

uint32_t stage_units(const rf_ctx *c, uint32_t nl, int stage, uint32_t chunk, bool small) {
    const uint32_t chunks = c->n / kEw;
    const uint32_t dn = (nl + c->alpha - 1) / c->alpha;
    const bool fused = modup_fused(c, true);
    const uint32_t ext = c->modup_levels[nl].ext_limbs;
    switch (stage) {
        case kTensor: return 0;  // formed by the INTT of d2 and the inner product
        case kInttD0: case kInttD1: return limb_units(c, nl, c->q_order[nl].n_wide, 1, small);
        case kModupConv: return fused ? 0 : dn * modup_chunks(nl, c->K, chunk) * chunks;
        case kNttExt0:
            return fused ? c->modup_units[nl].n * (c->n / kMixTile) : limb_units(c, ext, ext, 1, small);
        case kNttExt1: return limb_units(c, ext, c->ext_order[nl].n_wide, 1, small);
        case kInnerProduct: return (nl + c->K) * chunks;
        case kInttP0: case kInttP1: return limb_units(c, c->K, c->p_order.n_wide, 2, small);
        case kModdownConv: return 0;  // computed in the first pass of NTT(conv)
        case kNttConv0:
            return c->fp_mask.any() || small ? 2 * c->moddown_units[nl].n * (c->n / kMixTile) : 2 * nl * (c->n / kTile);
        case kNttConv1: return limb_units(c, nl, c->q_order[nl].n_wide, 2, small);
        case kTail: return 0;  // applied by the last pass of NTT(conv)
    }
    return 0;
}

int enqueue(rf_batch *p, hipStream_t s, bool profile) {
    static const char *names[kStages] = {"batch_tensor", "batch_ntt_inv_rows_tensor", "batch_ntt_inv_cols",
                                         "batch_modup_bconv", "batch_ntt_fwd_cols", "batch_ntt_fwd_rows",
                                         "batch_inner_product", "batch_ntt_inv_rows", "batch_ntt_inv_cols",
                                         "batch_moddown_bconv", "batch_ntt_fwd_cols_moddown", "batch_ntt_fwd_rows_moddown",
                                         "batch_moddown_tail"};
    for (int st = 0; st < kStages; ++st) {
        const uint32_t total = p->total[st];
        if (total == 0) continue;
        ProfScope prof(profile ? names[st] : nullptr, s);
        const bool ntt_step = st != kModupConv && st != kInnerProduct;
        if (!ntt_step) {
            const uint32_t g = p->grid[st] == 0 ? total : std::min(total, p->grid[st]);
            const uint32_t per = (total + g - 1) / g;
            const uint32_t blocks = (total + per - 1) / per;
            const uint32_t nj = p->n_items;
            switch (st) {
                case kModupConv:
                    if (p->modup_chunk == 4)
                        hipLaunchKernelGGL((ks_batched_kernel<kModupConv, 4>), blocks, kEw, 0, s, p->d_jobs, nj, total, per);
                    else if (p->modup_chunk == 16)
                        hipLaunchKernelGGL((ks_batched_kernel<kModupConv, 16>), blocks, kEw, 0, s, p->d_jobs, nj, total, per);
                    else
                        hipLaunchKernelGGL((ks_batched_kernel<kModupConv, 8>), blocks, kEw, 0, s, p->d_jobs, nj, total, per);
                    break;
                case kInnerProduct: hipLaunchKernelGGL(ks_batched_kernel<kInnerProduct>, blocks, kEw, 0, s, p->d_jobs, nj, total, per); break;
            }
        } else {
            // one launch per ring degree; the step's workgroups are shared out in
            // proportion to the units of each degree
            for (const rf_batch::Group &G : p->groups) {
                const uint32_t units = G.units[st];
                if (units == 0) continue;
                uint32_t g = units;
                if (p->grid[st] != 0)
                    g = std::max(1u, std::min(units, (uint32_t)(((uint64_t)p->grid[st] * units + total - 1) / total)));
                const uint32_t per = (units + g - 1) / g;
                const uint32_t blocks = (units + per - 1) / per;
                const NttJob *jobs = p->d_ntt[list_of(st)] + G.job0;
                const uint32_t nj = G.job1 - G.job0, u0 = G.unit0[st];
#define RF_BLK(A, B, PASS)                                                                                       \
    if (per == 1 && G.wide)                                                                                      \
        hipLaunchKernelGGL((ntt_batched_kernel<A, B, PASS, false, NoFp>), blocks, kThreads, 0, s, jobs, nj, u0, units, per); \
    else if (per == 1)                                                                                           \
        hipLaunchKernelGGL((ntt_batched_kernel<A, B, PASS, false, FpMask>), blocks, kThreads, 0, s, jobs, nj, u0, units, per); \
    else                                                                                                         \
        hipLaunchKernelGGL((ntt_batched_kernel<A, B, PASS, true, FpMask>), blocks, kThreads, 0, s, jobs, nj, u0, units, per)
#define RF_BL(A, B)                                                                                              \
    switch (st) {                                                                                                \
        case kInttD0: RF_BLK(A, B, kPassTensor); break;                                                          \
        case kInttP0: RF_BLK(A, B, kPassInvRows); break;                                                         \
        case kInttD1: case kInttP1: RF_BLK(A, B, kPassInvCols); break;                                           \
        case kNttExt0: RF_BLK(A, B, kPassModup); break;                                                          \
        case kNttExt1: RF_BLK(A, B, kPassFwdRows); break;                                                        \
        case kNttConv0:                                                                                          \
            if (G.k4) {                                                                                          \
                RF_BLK(A, B, kPassModdown4);                                                                     \
            } else {                                                                                             \
                RF_BLK(A, B, kPassModdown8);                                                                     \
            }                                                                                                    \
            break;                                                                                               \
        case kNttConv1: RF_BLK(A, B, kPassTail); break;                                                          \
    }
                switch (G.log_n) {
                    case 16: RF_BL(8, 8) break;
                    case 15: RF_BL(8, 7) break;
                    case 14: RF_BL(7, 7) break;
                    default: RF_BL(7, 6) break;
                }
#undef RF_BL
#undef RF_BLK
            }
        }
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return fail(RF_EHIP, std::string("batched launch: ") + hipGetErrorString(e));
    }
    return RF_OK;
}

void drop_graph(rf_batch *p) {
    if (p->exec) (void)hipGraphExecDestroy(p->exec);
    if (p->graph) (void)hipGraphDestroy(p->graph);
    p->exec = nullptr;
    p->graph = nullptr;
}

// Job tables of a plan from its items, workspace and ModUp chunk: the
// element-wise jobs, the four NTT job lists and the ring-degree groups.
void build_tables(rf_batch *p, std::vector<KsJob> &jobs, std::vector<NttJob> (&ntt)[4]) {
    const rf_batch_item *items = p->items.data();
    const uint32_t n = (uint32_t)p->items.size();
    jobs.assign(n, KsJob{});
    for (auto &v : ntt) v.assign(n, NttJob{});
    uint32_t acc[kStages] = {0};
    uint64_t *w = p->ws;
    // items in order of ring degree (the NTT steps run one launch per degree)
    std::vector<uint32_t> order(n);
    for (uint32_t i = 0; i < n; ++i) order[i] = i;
    std::stable_sort(order.begin(), order.end(),
                     [&](uint32_t x, uint32_t y) { return items[x].ctx->log_n < items[y].ctx->log_n; });
    // the tiles of the wide limbs of each launch
    bool small[17][4] = {};
    for (uint32_t ln = 13; ln <= 16; ++ln)
        for (int k = 0; k < 4; ++k) {
            uint64_t wide = 0, all = 0;  // 4096-residue tiles
            for (uint32_t i = 0; i < n; ++i) {
                const rf_ctx *c = items[i].ctx;
                if (c->log_n != ln) continue;
                const uint32_t nl = items[i].n_limbs, tiles = c->n / kTile;
                const uint32_t limbs[4] = {nl, c->modup_levels[nl].ext_limbs, 2 * c->K, 2 * nl};
                const uint32_t nw[4] = {c->q_order[nl].n_wide, c->ext_order[nl].n_wide, 2 * c->p_order.n_wide,
                                        2 * c->q_order[nl].n_wide};
                wide += (uint64_t)nw[k] * tiles;
                all += (uint64_t)limbs[k] * tiles;
            }
            small[ln][k] = batch_small(k, wide, all);
        }
    std::vector<rf_batch::Group> groups;
    for (uint32_t i = 0; i < n; ++i) {
        const rf_batch_item &it = items[order[i]];
        const rf_ctx *c = it.ctx;
        if (groups.empty() || groups.back().log_n != c->log_n) {
            if (!groups.empty()) {
                groups.back().job1 = i;
                for (int st = 0; st < kStages; ++st) groups.back().units[st] = acc[st] - groups.back().unit0[st];
            }
            rf_batch::Group G{};
            G.log_n = c->log_n;
            G.job0 = i;
            G.k4 = G.wide = true;
            for (int st = 0; st < kStages; ++st) G.unit0[st] = acc[st];
            groups.push_back(G);
        }
        if (c->K != 4) groups.back().k4 = false;
        if (c->fp_mask.any()) groups.back().wide = false;
        const uint32_t nl = it.n_limbs;
        const size_t N = c->n;
        const ModupLevel &lv = c->modup_levels[nl];
        KsJob &J = jobs[i];
        J.a = it.a;
        J.b = it.b;
        J.evk = it.rlk;
        J.out = it.out;
        J.d_coeff = w;
        J.ext = J.d_coeff + (size_t)nl * N;
        J.ip = J.ext + (size_t)lv.ext_limbs * N;
        J.conv = J.ip + 2 * (size_t)(nl + c->K) * N;
        w = J.conv + 2 * (size_t)nl * N;
        J.pcs = c->d_pc;
        J.modup_tab = c->d_modup;
        J.modup_stride = c->modup_stride;
        const uint64_t *moddown_tab = c->scheme == RF_BGV ? c->d_moddown_t : c->d_moddown;
        J.pinv = c->d_moddown + moddown_pinv_off(c);
        J.log_n = c->log_n;
        J.nl = nl;
        J.L = c->L;
        J.K = c->K;
        J.alpha = c->alpha;
        for (int st = 0; st < kStages; ++st) {
            J.unit_begin[st] = acc[st];
            acc[st] += stage_units(c, nl, st, p->modup_chunk, small[c->log_n][list_of(st)]);
        }
        const uint64_t ipstride = (uint64_t)(nl + c->K) * N;
        NttBatch bd{J.d_coeff, J.d_coeff, 0, 0, nl, 1, 0, nullptr, c->order(c->q_order[nl])};
        NttBatch be{J.ext, J.ext, 0, 0, lv.ext_limbs, 1, 0, nullptr, c->order(c->ext_order[nl])};
        NttBatch bp{J.ip + (size_t)nl * N, J.ip + (size_t)nl * N, ipstride, ipstride, c->K, 2, c->L, nullptr,
                    c->order(c->p_order)};
        NttBatch bc{J.conv, J.conv, (uint64_t)nl * N, (uint64_t)nl * N, nl, 2, 0, nullptr, c->order(c->q_order[nl])};
        const NttBatch bs[4] = {bd, be, bp, bc};
        const int first_stage[4] = {kInttD0, kNttExt0, kInttP0, kNttConv0};
        for (int k = 0; k < 4; ++k) {
            ntt[k][i].b = bs[k];
            ntt[k][i].tw_all = (k == 1 || k == 3) ? c->d_tw_fwd : c->d_tw_inv;
            ntt[k][i].tw_rows = (k == 1 || k == 3) ? c->d_tw_fwd_rows : c->d_tw_inv_rows;
            // the INTT of d2 folds the ModUp input factor, the INTT of the P-limbs the
            // ModDown input factor into its last stage
            ntt[k][i].pcs = k == 0 ? pc_modup(c, nl) : k == 2 ? c->d_pc_md : c->d_pc;
            ntt[k][i].log_n = c->log_n;
            for (int pass = 0; pass < 2; ++pass) ntt[k][i].unit_begin[pass] = J.unit_begin[first_stage[k] + pass];
            ntt[k][i].small = small[c->log_n][k];
            if (k == 1 && modup_fused(c, true)) {
                ntt[k][i].units = c->d_units + c->modup_units[nl].off;
                ntt[k][i].frag = c->d_conv_mu;
                ntt[k][i].off = c->d_conv_mu_off;
            } else if (k == 3 && (c->fp_mask.any() || small[c->log_n][k])) {
                ntt[k][i].units = c->d_units + c->moddown_units[nl].off;
                ntt[k][i].frag = c->d_conv_md;
                ntt[k][i].off = c->d_conv_md_off;
            }
            ntt[k][i].x = J.d_coeff;
            ntt[k][i].modup_tab = J.modup_tab;
            ntt[k][i].modup_stride = J.modup_stride;
            ntt[k][i].alpha = c->alpha;
            ntt[k][i].ct_a = it.a;
            ntt[k][i].ct_b = it.b;
            ntt[k][i].ip = J.ip;
            ntt[k][i].out = J.out;
            ntt[k][i].pinv = J.pinv;
            ntt[k][i].md_cross = moddown_tab + moddown_cross_off(c);
            ntt[k][i].md_negp = moddown_tab + moddown_negp_off(c);
            ntt[k][i].nl = nl;
            ntt[k][i].K = c->K;
            ntt[k][i].L = c->L;
        }
    }
    groups.back().job1 = n;
    for (int st = 0; st < kStages; ++st) groups.back().units[st] = acc[st] - groups.back().unit0[st];
    p->groups = groups;
    for (int st = 0; st < kStages; ++st) p->total[st] = acc[st];
}

// Rebuild and upload the job tables (the device buffers exist already).
int upload_tables(rf_batch *p) {
    std::vector<KsJob> jobs;
    std::vector<NttJob> ntt[4];
    build_tables(p, jobs, ntt);
    const uint32_t n = p->n_items;
    int prev = 0;
    (void)hipGetDevice(&prev);
    (void)hipSetDevice(p->device);
    // a launch of the plan still in flight reads the old tables
    bool ok = hipDeviceSynchronize() == hipSuccess &&
              hipMemcpy(p->d_jobs, jobs.data(), sizeof(KsJob) * n, hipMemcpyHostToDevice) == hipSuccess;
    for (int k = 0; k < 4 && ok; ++k)
        ok = hipMemcpy(p->d_ntt[k], ntt[k].data(), sizeof(NttJob) * n, hipMemcpyHostToDevice) == hipSuccess;
    (void)hipSetDevice(prev);
    return ok ? RF_OK : fail(RF_EHIP, "batch plan: upload of the job tables");
}

}  // namespace

extern "C" size_t rf_batch_workspace_bytes(const rf_batch_item *items, uint32_t n) {
    if (validate(items, n)) return 0;
    size_t limbs = 0;
    for (uint32_t i = 0; i < n; ++i) limbs += item_ws_limbs(items[i].ctx, items[i].n_limbs) * items[i].ctx->n;
    return limbs * 8;
}

extern "C" int rf_batch_create(const rf_batch_item *items, uint32_t n, void *ws, size_t ws_bytes, rf_batch **out) {
    int rc;
    if (!out) return fail(RF_EINVAL, "rf_batch_create: null out");
    *out = nullptr;
    if ((rc = validate(items, n))) return rc;
    const size_t need = rf_batch_workspace_bytes(items, n);
    if (!ws || ws_bytes < need)
        return fail(RF_EWORKSPACE, "rf_batch_create: workspace of " + std::to_string(ws_bytes) + " bytes, need " +
                                       std::to_string(need));
    rf_batch *p = new rf_batch();
    p->device = items[0].ctx->device;
    p->n_items = n;
    p->items.assign(items, items + n);
    p->ws = (uint64_t *)ws;
    int prev = 0;
    (void)hipGetDevice(&prev);
    (void)hipSetDevice(p->device);
    bool ok = hipMalloc((void **)&p->d_jobs, sizeof(KsJob) * n) == hipSuccess;
    for (int k = 0; k < 4 && ok; ++k) ok = hipMalloc((void **)&p->d_ntt[k], sizeof(NttJob) * n) == hipSuccess;
    (void)hipSetDevice(prev);
    if (!ok || upload_tables(p) != RF_OK) {
        rf_batch_destroy(p);
        return fail(RF_EHIP, "rf_batch_create: allocation or upload of the job tables");
    }
    *out = p;
    return RF_OK;
}

extern "C" void rf_batch_destroy(rf_batch *p) {
    if (!p) return;
    int prev = 0;
    (void)hipGetDevice(&prev);
    (void)hipSetDevice(p->device);
    drop_graph(p);
    if (p->capture_stream) (void)hipStreamDestroy(p->capture_stream);
    (void)hipFree(p->d_jobs);
    for (auto *d : p->d_ntt) (void)hipFree(d);
    (void)hipSetDevice(prev);
    delete p;
}

extern "C" int rf_batch_set_grid(rf_batch *p, uint32_t stage, uint32_t workgroups) {
    if (!p || stage >= (uint32_t)kStages) return fail(RF_EINVAL, "rf_batch_set_grid: bad stage");
    if (p->grid[stage] != workgroups) {
        p->grid[stage] = workgroups;
        drop_graph(p);
    }
    return RF_OK;
}

extern "C" int rf_batch_set_modup_chunk(rf_batch *p, uint32_t chunk) {
    if (!p) return fail(RF_EINVAL, "rf_batch_set_modup_chunk: null plan");
    if (chunk != 4 && chunk != 8 && chunk != 16) return fail(RF_EINVAL, "rf_batch_set_modup_chunk: 4, 8 or 16");
    if (p->modup_chunk == chunk) return RF_OK;
    p->modup_chunk = chunk;
    drop_graph(p);
    return upload_tables(p);
}

extern "C" int rf_batch_stage_units(const rf_batch *p, uint32_t stage) {
    if (!p || stage >= (uint32_t)kStages) return fail(RF_EINVAL, "rf_batch_stage_units: bad stage");
    return (int)p->total[stage];
}

extern "C" int rf_batch_hmult_relin(rf_batch *p, void *stream) {
    if (!p) return fail(RF_EINVAL, "rf_batch_hmult_relin: null plan");
    int prev = 0;
    (void)hipGetDevice(&prev);
    if (prev != p->device) (void)hipSetDevice(p->device);
    int rc = enqueue(p, (hipStream_t)stream, true);
    if (prev != p->device) (void)hipSetDevice(prev);
    return rc;
}

extern "C" int rf_batch_graph_launch(rf_batch *p, void *stream) {
    if (!p) return fail(RF_EINVAL, "rf_batch_graph_launch: null plan");
    int prev = 0;
    (void)hipGetDevice(&prev);
    if (prev != p->device) (void)hipSetDevice(p->device);
    int rc = RF_OK;
    if (!p->exec) {
        if (!p->capture_stream && hipStreamCreateWithFlags(&p->capture_stream, hipStreamNonBlocking) != hipSuccess)
            rc = fail(RF_EHIP, "rf_batch_graph_launch: stream");
        if (!rc && hipStreamBeginCapture(p->capture_stream, hipStreamCaptureModeThreadLocal) != hipSuccess)
            rc = fail(RF_EHIP, "rf_batch_graph_launch: begin capture");
        if (!rc) {
            int erc = enqueue(p, p->capture_stream, false);
            hipGraph_t g = nullptr;
            hipError_t e = hipStreamEndCapture(p->capture_stream, &g);
            if (erc) rc = erc;
            else if (e != hipSuccess || !g) rc = fail(RF_EHIP, "rf_batch_graph_launch: end capture");
            else {
                p->graph = g;
                if (hipGraphInstantiate(&p->exec, p->graph, nullptr, nullptr, 0) != hipSuccess) {
                    drop_graph(p);
                    rc = fail(RF_EHIP, "rf_batch_graph_launch: instantiate");
                }
            }
            if (rc && g && !p->graph) (void)hipGraphDestroy(g);
        }
    }
    if (!rc && hipGraphLaunch(p->exec, (hipStream_t)stream) != hipSuccess)
        rc = fail(RF_EHIP, "rf_batch_graph_launch: launch");
    if (prev != p->device) (void)hipSetDevice(prev);
    return rc;
}
