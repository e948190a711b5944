// Internal structures of the RNS-FHE library shared by the host runtime and the kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>
#include <vector>

#include "../../include/rnsfhe.h"

namespace rf {

constexpr int kMaxAlpha = 8;
constexpr int kMaxBfvLimbs = 24;  // BFV: Q-primes and auxiliary primes the BEHZ kernels hold in registers
constexpr uint32_t kMaxCrtLimbs = 32;  // limbs of a CRT composition
constexpr int kMaxPrimes = 250;  // L + k, prime indices fit in a byte

// Per-prime constants, device resident.  Prime index g < L is q_g, g >= L is p_{g-L}.
struct PrimeConst {
    uint64_t q;
    uint64_t mu1, mu0;       // floor(2^128 / q) = mu1 * 2^64 + mu0
    uint64_t ninv, ninv_p;   // N^-1 mod q and its Shoup companion
    uint64_t wlast, wlast_p; // psi^-brv(1) * N^-1 (last inverse stage) and companion
    uint64_t tmod, tmod_p;   // plaintext modulus t mod q and companion (BGV/BFV; 0 for CKKS)
    uint64_t tinv, tinv_p;   // t^-1 mod q and companion
    uint64_t r64, r64_p;     // 2^64 mod q and companion
    uint64_t one_p;          // floor(2^64 / q): Shoup companion of 1
    double qd, qinv;         // q and 1 / q in FP64 (primes below kFpPrimeBound; see FpMod)
};

// Twiddles.  A prime's table takes N pairs of memory; a prime below
// kFpPrimeBound keeps N doubles (the twiddles in [-q/2, q/2]) at its start
// instead: FP64 products need no companion, so a pass reads half the bytes.
struct __align__(16) TwPair {
    uint64_t w, wp;  // twiddle and floor(w 2^62 / q) (the companion of shoup62_lazy)
};

// Which primes are below kFpPrimeBound, one bit per prime index, passed to the
// kernels by value: the arithmetic of a limb is then known from the kernel
// arguments, so its loads need not wait for the prime's constants to arrive.
struct FpMask {
    uint64_t m[4];
    __host__ __device__ __forceinline__ bool has(uint32_t g) const {
        const uint64_t w = g < 128 ? (g < 64 ? m[0] : m[1]) : (g < 192 ? m[2] : m[3]);
        return (w >> (g & 63)) & 1;
    }
    bool any() const { return (m[0] | m[1] | m[2] | m[3]) != 0; }
};
// The mask of a launch with no such prime (chains of wide primes, and the wide limbs
// of any other on their own): its kernels hold the integer code alone.  With both
// forms in every kernel the few-limb passes of a chain of 55-bit primes took 2.5 %
// longer (HMult+Relin of 9 limbs at N = 2^15, 115.6 against 112.4 us).
struct NoFp {
    __host__ __device__ __forceinline__ static constexpr bool has(uint32_t) { return false; }
};
// A transform of wide primes alone, many limbs: 4096-residue tiles (ntt.hip).
struct WideTiles {};

// The limbs of a launch with those of wide primes first: device entries limb |
// prime << 16, n_wide of them wide.  A window of the chain is two runs of the
// whole chain's order, its wide primes and, gap entries further on, its narrow
// ones; base is its first limb (both 0 for an order of its own).  A launch has fewer
// than 65536 limbs, a chain at most kMaxPrimes.  16 bytes: with 24 the kernels'
// arguments ran into another cache line, 0.3 to 0.9 us a launch.  Bit-fields, not
// smaller members: scalar loads read whole words, and a batch's kernels, which take
// this from memory, held a 16-bit n_wide in vector registers (the last row pass of
// 20 items at N = 2^16 4 spills, 238.6 us against 227.7).
struct LimbOrder {
    const uint32_t *ent;
    uint32_t n_wide : 16, gap : 8, base : 8;
};
static_assert(sizeof(LimbOrder) == 16, "a launch's arguments");

// Launch description of a batched (I)NTT over limbs laid out as
// [n_polys][per_poly][N]; limb i of a polynomial uses prime pmap[i] (or prime_base + i).
struct NttBatch {
    const uint64_t *in;
    uint64_t *out;
    uint64_t in_poly_stride;   // elements between polynomials
    uint64_t out_poly_stride;
    uint32_t per_poly;
    uint32_t n_polys;
    uint32_t prime_base;
    const uint32_t *pmap;      // device array [per_poly] or nullptr
    LimbOrder order{};         // the same limbs in launch order
    bool blocked = false;      // the coefficient side is in the blocked layout (ntt_dev.hpp)
};

// Offsets (uint64 entries) of the BEHZ tables of a BFV context (L Q-primes,
// nb auxiliary primes B, B_sk = B u {m_sk}, m~ = 2^32).  The constants of one
// output limb of a conversion are contiguous (target-major), so a thread reads
// them with wide scalar loads.
struct BehzLayout {
    uint32_t L, nb;
    uint32_t ext_factor;   // [L] pairs: m~ (Q/q_i)^-1 mod q_i
    uint32_t ext_cross;    // [nb+1][L]: (Q/q_i) m~^-1 mod bsk_m
    uint32_t ext_q;        // [nb+1] pairs: Q m~^-1 mod bsk_m
    uint32_t cross_q_mt;   // [L]: Q/q_i mod 2^32
    uint32_t neg_qinv_mt;  // [1]: -Q^-1 mod 2^32
    uint32_t floor_factor; // [L] pairs: t (Q/q_i)^-1 mod q_i
    uint32_t floor_cross;  // [nb+1][L]: Q/q_i mod bsk_m
    uint32_t t_bsk;        // [nb+1] pairs: t mod bsk_m
    uint32_t qinv_bsk;     // [nb+1] pairs: Q^-1 mod bsk_m
    uint32_t sk_factor;    // [nb] pairs: (M/b_j)^-1 mod b_j
    uint32_t sk_cross;     // [L][nb]: M/b_j mod q_i
    uint32_t cross_b_msk;  // [nb]: M/b_j mod m_sk
    uint32_t minv_msk;     // [1] pair: M^-1 mod m_sk
    uint32_t m_q;          // [L] pairs: M mod q_i
    uint32_t total;
};

// Host-side layout of the ModUp extension basis at one level.
struct ModupLevel {
    uint32_t dnum;        // digits at this level
    uint32_t ext_limbs;   // sum over digits of (nl - alpha_j + k)
    uint32_t pmap_off;    // offset of this level's prime map in Context::d_pmaps
};

// The targets one workgroup of a fused base conversion takes (convert.hip): one
// limb of a wide prime, or up to four of narrow ones.
struct ConvUnit {
    uint32_t digit, size;  // ModUp: the digit and its number of primes
    uint32_t count, wide;
    uint32_t e[4];         // limb | prime << 16, the last one repeated from count on
};

// Constants of a conversion as the matrix instruction's operand (convert.hip):
// per block (ModUp: modup_block's order; ModDown: one) and target prime g the
// bytes [8][kp][8] at (block * primes + g) * conv_bytes(kp), kp = 4 or 8 sources,
// and off[block * primes + g].
inline uint32_t conv_kp(uint32_t sources) { return sources <= 4 ? 4 : 8; }
inline size_t conv_bytes(uint32_t kp) { return 64 * (size_t)kp; }

}  // namespace rf

struct rf_ctx {
    int device;
    int scheme;
    uint32_t log_n, log_nmax, n;
    uint32_t L, K, alpha, dnum;
    uint64_t t;
    std::vector<uint64_t> primes;  // L + K: q_0..q_{L-1}, p_0..p_{k-1}
    std::vector<uint64_t> psi;     // primitive 2N-th roots
    rf::FpMask fp_mask{};          // primes below rf::kFpPrimeBound
    std::vector<rf::ModupLevel> modup_levels;  // index nl in [1, L]
    std::vector<rf_tuning> tuning;             // kernel variants per level nl in [1, L] (index 0 unused)

    // device tables (owned)
    rf::PrimeConst *d_pc = nullptr;        // [L+K]
    rf::PrimeConst *d_pc_md = nullptr;     // d_pc with the ModDown input factor [(P/p_a)^-1]_{p_a}
                                           // folded into the last inverse stage of every special prime
    rf::PrimeConst *d_pc_mu = nullptr;     // [L][L+K]: per level nl (row nl - 1), d_pc with the ModUp
                                           // input factor [(Q_j/q_i)^-1]_{q_i} of limb i < nl (digit j
                                           // at that level) folded into its last inverse stage
    rf::TwPair *d_tw_fwd = nullptr;        // [L+K][N]: psi^brv(k)
    rf::TwPair *d_tw_inv = nullptr;        // [L+K][N]: psi^-brv(k)
    rf::TwPair *d_tw_fwd_rows = nullptr;   // the same twiddles in the row-pass layout (ntt_dev.hpp)
    rf::TwPair *d_tw_inv_rows = nullptr;
    uint64_t *d_modup = nullptr;           // ModUp base-conversion constants, see context.hip
    uint64_t *d_moddown = nullptr;         // ModDown constants
    uint64_t *d_moddown_t = nullptr;       // ModDown constants keeping the message mod t (BGV)
    uint64_t *d_rescale = nullptr;         // rescale constants
    uint32_t *d_pmaps = nullptr;           // ModUp extension prime maps for every level
    uint32_t *d_order = nullptr;           // rf::LimbOrder entries of the windows below
    struct OrderRef {
        uint32_t off = 0, n_wide = 0;
    };
    std::vector<OrderRef> q_order, ext_order;  // index nl: q_0..q_{nl-1}; the ModUp extension
    OrderRef p_order, all_order, qb_order;     // the special primes; Q u P; q u B_sk (BFV)
    struct UnitRef {
        uint32_t off = 0, n = 0;
    };
    std::vector<UnitRef> modup_units, moddown_units;  // index nl: rf::ConvUnit windows of d_units
    rf::ConvUnit *d_units = nullptr;
    // narrow targets' conversion constants (null without narrow primes): ModUp, ModDown (BGV: t's)
    int8_t *d_conv_mu = nullptr, *d_conv_md = nullptr;
    double *d_conv_mu_off = nullptr, *d_conv_md_off = nullptr;
    rf::LimbOrder order(const OrderRef &r) const { return rf::LimbOrder{d_order + r.off, (uint16_t)r.n_wide, 0, 0}; }
    // BFV: auxiliary base B and m_sk follow the special primes in `primes`
    uint32_t nb = 0;
    uint64_t *d_behz = nullptr;            // BEHZ tables (rf::BehzLayout)
    uint32_t *d_pmap_qb = nullptr;         // prime indices of q u B_sk
    rf::BehzLayout behz{};
    size_t modup_stride = 0;               // uint64 entries per (digit, size) block
    // client side (key generation, encryption, decryption, encode / decode)
    uint64_t *d_client = nullptr;          // [L+K][4]: [P]_{p_g}, companion, [floor(Q_L / t)]_{p_g} (BFV), companion
    uint64_t *d_garner = nullptr;          // [L][L][2]: (q_i^-1 mod q_j, companion) for i < j
    double *d_garner_fp = nullptr;         // [L + 32] pairs (q_j, 1 / q_j), then [L][L + 32]: q_i^-1 mod q_j in
                                           // (-q_j/2, q_j/2), q_j below kFpPrimeBound; the last 32 columns padding
    double *d_zeta = nullptr;              // CKKS: [2N][2] (cos, sin)(pi k / N)
    uint32_t *d_slot_of = nullptr;         // CKKS: [N] the slot j with 5^j = 2t + 1 mod 2N, or j | 2^31 with -5^j = 2t + 1
};

namespace rf {

// Defaults of rf_tuning.
constexpr rf_tuning kDefaultTuning = {256, 0, 4, 8, 0};
inline const rf_tuning &level_tuning(const rf_ctx *c, uint32_t nl) {
    return c->tuning[nl < 1 ? 1 : (nl > c->L ? c->L : nl)];
}

// What the inner product adds on the Q-limbs when the ModDown tail that follows
// is reduced to out = ip' - NTT(conv) P^-1 (the fused two-pass path):
// ip'[c][m] = ip[c][m] P^-1 + add_c[m].  pinv null: the plain inner product.
struct IpFold {
    const uint64_t *pinv = nullptr;  // pairs (P^-1 mod q_i, companion)
    // Where the digit's own residue d[m] and the addends come from:
    //   0: d and add0/add1 (nullable) as given;
    //   1 (HMult+Relin): a, b = [2][nl][N] ciphertexts in the NTT domain:
    //      d = a1 b1, add0 = a0 b0, add1 = a0 b1 + a1 b0 (the tensor), computed here;
    //   2 (HRotate): a = the input ciphertext: d = sigma_g(a1), add0 = sigma_g(a0)
    //      (g = galois), gathered here; no add1.
    uint32_t mode = 0;
    const uint64_t *add0 = nullptr, *add1 = nullptr;
    const uint64_t *a = nullptr, *b = nullptr;
    uint32_t galois = 0;
};

// Index map of sigma_g in the NTT domain (output k holds a(psi^(2 brv(k) + 1))):
// sigma_g(a)[k] = a[k'] with 2 brv(k') + 1 = (2 brv(k) + 1) g mod 2N.
__device__ __forceinline__ uint32_t galois_src(uint32_t k, uint32_t galois, uint32_t log_n) {
    const uint32_t mask2n = (2u << log_n) - 1;
    const uint32_t rk = __brev(k) >> (32 - log_n);
    const uint32_t e = ((2u * rk + 1u) * galois) & mask2n;
    return __brev((e - 1u) >> 1) >> (32 - log_n);
}

// Offsets (in uint64 entries) inside the ModUp table block of (digit j, digit size s):
//   [0, 2*alpha):            factor pairs (w, w') of [(Q_j/q_i)^-1]_{q_i}, i' < s
//   [2*alpha, ...):          cross[g][i'] = [Q_j/q_i]_{prime g}, g in [0, L+K), target-major
inline size_t modup_block(const rf_ctx *c, uint32_t j, uint32_t s) {
    return ((size_t)j * c->alpha + (s - 1)) * c->modup_stride;
}
// INTT constants of level nl whose output is the ModUp input y_i = [x_i (Q_j/q_i)^-1]_{q_i}.
inline const PrimeConst *pc_modup(const rf_ctx *c, uint32_t nl) {
    return c->d_pc_mu + (size_t)(nl - 1) * (c->L + c->K);
}
// ModDown table: [K] factor pairs (w, w') of [(P/p)^-1]_p; [L][K] cross [P/p]_{q_i} (target-major);
// [L] pairs P^-1 mod q_i; [L] (q_i - [P]_{q_i}).
inline size_t moddown_cross_off(const rf_ctx *c) { return 2 * (size_t)c->K; }
inline size_t moddown_pinv_off(const rf_ctx *c) { return 2 * (size_t)c->K + (size_t)c->K * c->L; }
inline size_t moddown_negp_off(const rf_ctx *c) { return moddown_pinv_off(c) + 2 * (size_t)c->L; }
// Rescale table, per dropped prime index l in [1, L) and i < l:
//   entry (l * L + i) * 3 + {0,1,2} = q_l^-1 mod q_i, its companion, q_i - [q_l]_{q_i}.
inline size_t rescale_off(const rf_ctx *c, uint32_t l, uint32_t i) {
    return ((size_t)l * c->L + i) * 3;
}

// Brackets one kernel launch with HIP events on its stream while profiling is
// enabled (rf_profile_enable); a no-op otherwise.
class ProfScope {
  public:
    ProfScope(const char *name, hipStream_t s);
    ~ProfScope();

  private:
    int idx_;
    hipStream_t s_;
};

void set_error(const std::string &msg);
int fail(int code, const std::string &msg);

// kernel launchers (kernels.hip)
// pcs: per-prime constants (null: the context's d_pc).
// tn: the level's kernel variants (null: the defaults).
int launch_ntt(const rf_ctx *c, const NttBatch &b, bool forward, hipStream_t s, const PrimeConst *pcs = nullptr,
               const rf_tuning *tn = nullptr);
// First pass alone of the INTT of b's few limbs, into the blocked layout (contexts with narrow primes).
int launch_intt_rows(const rf_ctx *c, const NttBatch &b, hipStream_t s);
// Second pass alone of the INTT of b's limbs, in place (two-pass ring degrees).
// mixed: the kernel of both classes for limbs of wide primes alone too.
int launch_intt_cols(const rf_ctx *c, const NttBatch &b, hipStream_t s, const PrimeConst *pcs = nullptr,
                     const rf_tuning *tn = nullptr, bool mixed = false);
// Last pass alone of the forward NTT of b's limbs after launch_modup_cols.
int launch_ntt_fwd_rows(const rf_ctx *c, const NttBatch &b, hipStream_t s, const rf_tuning *tn);
// ModUp conversion and the first pass of the extension's NTT in one launch
// (convert.hip): x [nl][N] as launch_modup_bconv's scaled input, ext its output
// after the column pass, both in the blocked layout or both not.  modup_fused:
// whether a key switch takes it.
bool modup_fused(const rf_ctx *c, bool scaled);
int launch_modup_cols(const rf_ctx *c, const uint64_t *x, uint64_t *ext, uint32_t nl, bool blocked, hipStream_t s);
// The first pass of NTT(conv) after the ModDown conversion, likewise (contexts with narrow primes).
int launch_moddown_cols(const rf_ctx *c, const uint64_t *ip, uint64_t *conv, uint32_t nl, hipStream_t s);
// ModDown after the inner product, two-pass ring degrees only: ip = [2][nl + K][N]
// whose K P-limbs hold the INTT with d_pc_md (so already scaled by the input
// factor; blocked layout).  The first forward pass computes the base conversion of each Q
// target in its prologue (into conv [2][nl][N]), the last applies the tail:
// out[c][i] = (ip[c][i] - NTT(conv)) P^-1 + add_c.
// ip's Q-limbs must come from launch_inner_product with fold (P^-1 and the addends
// applied), so the tail is out[c][i] = ip[c][i] - NTT(conv)[c][i] P^-1.
int launch_ntt_fwd_moddown(const rf_ctx *c, uint64_t *conv, const uint64_t *ip, uint64_t *out, uint32_t nl,
                           hipStream_t s, const rf_tuning *tn = nullptr);
// INTT of the polynomial to key-switch (two-pass ring degrees only), with the
// step that produces it as the prologue of its first pass, into dc [nl][N]
// (coefficient domain, blocked layout, scaled for ModUp by pc_modup(c, nl)):
//   galois == 0 (HMult): d2 = a1 b1 of a, b ([2][nl][N]);
//   galois != 0 (HRotate): sigma_g of a's polynomial 1.
int launch_intt_first(const rf_ctx *c, const uint64_t *a, const uint64_t *b, uint64_t *dc, uint32_t galois,
                      uint32_t nl, hipStream_t s, const rf_tuning *tn = nullptr);
// The last pass of the INTT of last, the lift and the first pass of NTT(lift).
// lift_fused: whether a division by the last of nl primes takes it.
bool lift_fused(const rf_ctx *c, uint32_t nl);
int launch_lift_cols(const rf_ctx *c, const uint64_t *last, uint64_t *lift, uint32_t nl, bool keep_t, hipStream_t s);
// Rescale / modulus switch after the INTT of the last limb (last = [2][N],
// blocked; where lift_fused after its row pass only),
// two-pass ring degrees only: the first forward pass lifts the last limb into
// each remaining prime in its prologue (into lift [2][nl-1][N]; KEEP_T for BGV),
// the last applies the tail out[c][i] = (in[c][i] - NTT(lift)) q_l^-1.
int launch_ntt_fwd_rescale(const rf_ctx *c, const uint64_t *last, uint64_t *lift, const uint64_t *in,
                           uint64_t *out, uint32_t nl, bool keep_t, hipStream_t s, const rf_tuning *tn = nullptr);
int launch_tensor(const rf_ctx *c, const uint64_t *a, const uint64_t *b, uint64_t *d01,
                  uint64_t *d2, uint32_t nl, hipStream_t s);
// scaled: x is an INTT taken with pc_modup(c, nl), so each limb already carries
// its digit's input factor [(Q_j/q_i)^-1]_{q_i}.
// chunk: output limbs per thread (4, 8 or 16).
int launch_modup_bconv(const rf_ctx *c, const uint64_t *x, uint64_t *ext, uint32_t nl, hipStream_t s,
                       bool scaled = false, uint32_t chunk = 8);
// The Q-limbs leave as ip P^-1 + add_c with the sources fold names (its pinv is
// filled in here), for launch_ntt_fwd_moddown; the P-limbs after the first pass
// of their INTT (launch_intt_cols follows; two-pass ring degrees only).
int launch_inner_product(const rf_ctx *c, const uint64_t *d_ntt, const uint64_t *ext, const uint64_t *evk, uint64_t *ip,
                         uint32_t nl, hipStream_t s, const IpFold &fold);

// N = 2^12: a workgroup holds a whole limb, so a step that precedes or follows
// a transform needs no launch of its own (single.hip).
int launch_ntt_single(const rf_ctx *c, const NttBatch &b, bool forward, hipStream_t s, const PrimeConst *pcs);
// A key switch after fold's sources (its pinv is filled in here): INTT of the
// polynomial to switch (coef non-null: its coefficients instead), ModUp with
// the NTT of the extension, inner product with the INTT of the special limbs,
// ModDown, into out [2][nl][N].  Scratch: dc [nl], ext, ip [2][nl + K] limbs.
int launch_keyswitch_single(const rf_ctx *c, const IpFold &fold, const uint64_t *d, const uint64_t *coef,
                            const uint64_t *evk, uint64_t *dc, uint64_t *ext, uint64_t *ip, uint64_t *out,
                            uint32_t nl, hipStream_t s);
// Rescale / modulus switch (keep_t: BGV) of in [2][nl][N] into out [2][nl-1][N].
int launch_divide_single(const rf_ctx *c, const uint64_t *in, uint64_t *out, uint32_t nl, bool keep_t, hipStream_t s);

int launch_ewise(const rf_ctx *c, int op, const uint64_t *a, const uint64_t *b, int64_t k, uint64_t *out,
                 uint32_t nl, uint32_t n_polys, hipStream_t s);
int launch_behz_extend(const rf_ctx *c, const uint64_t *a, const uint64_t *b, uint64_t *ext, hipStream_t s);
// BEHZ fast floor (into f [3][nb+1][N], scratch) and Shenoy-Kumaresan
// conversion of tens = [3][L+nb+1][N]: d0, d1 to out01 [2][L][N], d2 to out2 [L][N].
int launch_behz_floor_sk(const rf_ctx *c, const uint64_t *tens, uint64_t *f, uint64_t *out01, uint64_t *out2,
                         hipStream_t s);
int launch_tensor_map(const rf_ctx *c, const uint64_t *a, const uint64_t *b, uint64_t *d01, uint64_t *d2,
                      uint32_t nl, const uint32_t *pmap, hipStream_t s);
int launch_automorphism(const rf_ctx *c, const uint64_t *in, uint64_t *out, uint32_t galois,
                        uint32_t nl, uint32_t n_polys, hipStream_t s);

}  // namespace rf
