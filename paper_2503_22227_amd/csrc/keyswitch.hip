// Element-wise and base-conversion kernels of HMult+Relin, HRotate and rescale.
//
// All kernels are one thread per coefficient of one limb (grid.x covers N in
// blocks of 256, grid.y enumerates limbs or digits), read and write whole
// 128-byte lines per wavefront, and take their per-prime constants from the
// context tables; indices that are uniform across a workgroup (limb, digit,
// target prime) come from blockIdx so the compiler keeps them in SGPRs and
// reads the constants with scalar loads.
//
// Key switching is the hybrid method (the paper's relinearize/rotate rows do
// not name one):
//   ModUp        y_i = [x_i (Q_j/q_i)^-1]_{q_i},  out_m = sum_{i in D_j} y_i [Q_j/q_i]_m
//   inner prod.  (sum_j ext_j evk_{j,0}, sum_j ext_j evk_{j,1}) on Q_l u P
//   ModDown      y_p = [x_p (P/p)^-1]_p taken in (-p/2, p/2],
//                conv_i = sum_p y_p [P/p]_{q_i}, out_i = (x_i - NTT(conv_i)) P^-1
// Sums of products are accumulated exactly in 128 bits and reduced once.
#include <hip/hip_runtime.h>

#include "ks_dev.hpp"
#include "ntt_dev.hpp"

namespace rf {

__global__ __launch_bounds__(kEw) void tensor_kernel(const uint64_t *__restrict__ a, const uint64_t *__restrict__ b,
                                                     uint64_t *__restrict__ d01, uint64_t *__restrict__ d2,
                                                     const PrimeConst *__restrict__ pcs, uint32_t log_n, uint32_t nl,
                                                     const uint32_t *pmap) {
    tensor_unit(a, b, d01, d2, pcs, log_n, nl, pmap, blockIdx.x, blockIdx.y);
}

__global__ __launch_bounds__(kEw) void behz_extend_kernel(const uint64_t *a, const uint64_t *b, uint64_t *ext,
                                                          const PrimeConst *__restrict__ pcs,
                                                          const uint64_t *__restrict__ tab, BehzLayout o, uint32_t kb,
                                                          uint32_t log_n) {
    behz_extend_unit(a, b, ext, pcs, tab, o, kb, log_n, blockIdx.x, blockIdx.y);
}

__global__ __launch_bounds__(kEw) void behz_floor_kernel(const uint64_t *tens, uint64_t *f,
                                                         const PrimeConst *__restrict__ pcs,
                                                         const uint64_t *__restrict__ tab, BehzLayout o, uint32_t kb,
                                                         uint32_t log_n) {
    behz_floor_unit(tens, f, pcs, tab, o, kb, log_n, blockIdx.x, blockIdx.y);
}

__global__ __launch_bounds__(kEw) void behz_sk_kernel(const uint64_t *f, uint64_t *out01, uint64_t *out2,
                                                      const PrimeConst *__restrict__ pcs,
                                                      const uint64_t *__restrict__ tab, BehzLayout o, uint32_t kb,
                                                      uint32_t log_n) {
    behz_sk_unit(f, out01, out2, pcs, tab, o, kb, log_n, blockIdx.x, blockIdx.y);
}

template <bool SCALED, int CH>
__global__ __launch_bounds__(kEw) void modup_bconv_kernel(const uint64_t *__restrict__ x, uint64_t *__restrict__ ext,
                                                          const PrimeConst *__restrict__ pcs,
                                                          const uint64_t *__restrict__ tab, size_t tab_stride,
                                                          uint32_t log_n, uint32_t nl, uint32_t L, uint32_t K,
                                                          uint32_t alpha) {
    modup_bconv_unit<SCALED, CH>(x, ext, pcs, tab, tab_stride, log_n, nl, L, K, alpha, blockIdx.x, blockIdx.y);
}

// Inner product of a P-limb as the prologue of its INTT: E residues a thread,
// digit by digit.  The P-limbs lie in no digit, so every source is the extension's.
template <int E>
struct IpRowsPro {
    static constexpr bool kBlocked = false;
    const uint64_t *ext, *key;  // the limb in digit 0's extension and key
    size_t ext_step, key_step;  // from a digit to the next
    size_t short_step;          // what the last digit's limb lies further on (fewer of its own primes)
    uint32_t dn;
    uint64_t q, r64, r64_p, one_p;
    template <typename Ar>
    __device__ __forceinline__ void tile(typename Ar::V (&v)[E], size_t first, int step, const Ar &) const {
        u128 acc[E];
#pragma unroll
        for (int r = 0; r < E; ++r) acc[r] = u128{0, 0};
#pragma unroll 1
        for (uint32_t j = 0; j < dn; ++j) {
            const uint64_t *e = ext + j * ext_step + (j + 1 == dn ? short_step : 0) + first;
            const uint64_t *k = key + j * key_step + first;
#pragma unroll
            for (int r = 0; r < E; ++r) mac(acc[r], e[r * step], k[r * step]);
        }
#pragma unroll
        for (int r = 0; r < E; ++r) {
            const uint64_t x = csub(reduce128_lazy(acc[r], q, r64, r64_p, one_p), 2 * q);
            if constexpr (Ar::kFp) v[r] = FpMod::from_u52(x);
            else v[r] = x;
        }
    }
};
template <int E>
constexpr bool kTilePro<IpRowsPro<E>> = true;

// The inner product on Q_l u P with the first pass of the INTT of its P-limbs,
// which come first: (limb, polynomial, tile of 1024 residues) a workgroup; then
// 256 coefficients of a Q-limb each.  Bound by the keys' and the extension's bytes.
// At 64 registers the streaming part keeps its 8 waves on a SIMD (the P-limbs' part
// spills 6 to 12), and that pass costs no launch of its own: with it, N = 2^16, 24 + 4
// limbs, alpha = 8: 40.0 us against 35.2 + 6.4; 9 + 4 limbs, alpha = 4: 19.0 against
// 15.9 + 6.2; N = 2^13, 5 + 4 limbs 5.3 against 3.9 + 4.2.
template <int A, int B, typename Fp>
__global__ __launch_bounds__(kEw) __attribute__((amdgpu_waves_per_eu(8))) void inner_product_kernel(
    const uint64_t *__restrict__ d, const uint64_t *__restrict__ ext, const uint64_t *__restrict__ evk,
    uint64_t *__restrict__ ip, const PrimeConst *__restrict__ pcs, const TwPair *__restrict__ tw_inv, Fp fpm, uint32_t nl,
    uint32_t L, uint32_t K, uint32_t alpha, IpFold fold) {
    __shared__ uint64_t lds[(1 << B) * ((kMixTile >> B) + 1)];
    constexpr int LOGN = A + B, TL = LOGN - 10;
    const uint32_t np = 2 * K << TL;
    if (blockIdx.x >= np) {
        const uint32_t w = blockIdx.x - np;
        inner_product_unit<1>(d, ext, evk, ip, pcs, LOGN, nl, L, K, alpha, w & ((1u << (LOGN - 8)) - 1), w >> (LOGN - 8),
                              fold);
        return;
    }
    const uint32_t u = blockIdx.x >> TL, poly = u & 1, m = nl + (u >> 1), g = L + (u >> 1);
    const PrimeConst pc = pcs[g];
    const uint32_t dn = (nl + alpha - 1) / alpha, full = min(alpha, nl);
    IpRowsPro<kMixE> pro;
    pro.ext = ext + ((size_t)(m - full) << LOGN);
    pro.key = evk + (((size_t)poly * (L + K) + g) << LOGN);
    pro.ext_step = (size_t)(nl + K - alpha) << LOGN;
    pro.key_step = (size_t)2 * (L + K) << LOGN;
    pro.short_step = (size_t)(full - (nl - (dn - 1) * alpha)) << LOGN;
    pro.dn = dn;
    pro.q = pc.q;
    pro.r64 = pc.r64;
    pro.r64_p = pc.r64_p;
    pro.one_p = pc.one_p;
    ntt_rows_small_pe<A, B, false, kMixTile, kMixE>(lds, pro, tw_inv + ((size_t)g << LOGN), pc, fpm.has(g),
                                                    blockIdx.x & ((1u << TL) - 1),
                                                    BlkRawEpi{ip + (((size_t)poly * (nl + K) + m) << LOGN)});
}

__global__ __launch_bounds__(kEw) void automorphism_kernel(const uint64_t *__restrict__ in, uint64_t *__restrict__ out,
                                                           uint32_t galois, uint32_t log_n) {
    automorphism_unit(in, out, galois, log_n, blockIdx.x, blockIdx.y);
}

template <int OP>
__global__ __launch_bounds__(kEw) void ewise_kernel(const uint64_t *a, const uint64_t *b, int64_t k, uint64_t *out,
                                                    const PrimeConst *__restrict__ pcs, uint32_t log_n, uint32_t nl) {
    ewise_unit<OP>(a, b, k, out, pcs, log_n, nl, blockIdx.x, blockIdx.y);
}

static int check_launch(const char *what) {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(RF_EHIP, std::string(what) + ": " + hipGetErrorString(e));
    return RF_OK;
}

static dim3 ew_grid(const rf_ctx *c, uint32_t y) { return dim3(c->n / kEw, y); }

int launch_tensor(const rf_ctx *c, const uint64_t *a, const uint64_t *b, uint64_t *d01, uint64_t *d2, uint32_t nl,
                  hipStream_t s) {
    ProfScope prof("tensor", s);
    hipLaunchKernelGGL(tensor_kernel, ew_grid(c, nl), dim3(kEw), 0, s, a, b, d01, d2, c->d_pc, c->log_n, nl,
                       (const uint32_t *)nullptr);
    return check_launch("tensor");
}

int launch_tensor_map(const rf_ctx *c, const uint64_t *a, const uint64_t *b, uint64_t *d01, uint64_t *d2,
                      uint32_t nl, const uint32_t *pmap, hipStream_t s) {
    ProfScope prof("tensor", s);
    hipLaunchKernelGGL(tensor_kernel, ew_grid(c, nl), dim3(kEw), 0, s, a, b, d01, d2, c->d_pc, c->log_n, nl, pmap);
    return check_launch("tensor");
}

int launch_behz_extend(const rf_ctx *c, const uint64_t *a, const uint64_t *b, uint64_t *ext, hipStream_t s) {
    ProfScope prof("behz_extend", s);
    hipLaunchKernelGGL(behz_extend_kernel, ew_grid(c, 4 * behz_groups(c->nb + 1)), dim3(kEw), 0, s, a, b, ext, c->d_pc,
                       c->d_behz, c->behz,
                       c->L + c->K, c->log_n);
    return check_launch("behz_extend");
}

int launch_behz_floor_sk(const rf_ctx *c, const uint64_t *tens, uint64_t *f, uint64_t *out01, uint64_t *out2,
                         hipStream_t s) {
    const uint32_t kb = c->L + c->K;
    {
        ProfScope prof("behz_floor", s);
        hipLaunchKernelGGL(behz_floor_kernel, ew_grid(c, 3 * behz_groups(c->nb + 1)), dim3(kEw), 0, s, tens, f,
                           c->d_pc, c->d_behz, c->behz, kb, c->log_n);
    }
    ProfScope prof("behz_sk", s);
    hipLaunchKernelGGL(behz_sk_kernel, ew_grid(c, 3 * behz_groups(c->L)), dim3(kEw), 0, s, f, out01, out2, c->d_pc,
                       c->d_behz, c->behz, kb, c->log_n);
    return check_launch("behz_floor_sk");
}

int launch_modup_bconv(const rf_ctx *c, const uint64_t *x, uint64_t *ext, uint32_t nl, hipStream_t s, bool scaled,
                       uint32_t chunk) {
    const uint32_t dn = (nl + c->alpha - 1) / c->alpha;
    if (chunk != 4 && chunk != 8 && chunk != 16) return fail(RF_EINVAL, "modup_bconv: chunk of 4, 8 or 16 limbs");
    ProfScope prof("modup_bconv", s);
    const dim3 grid = ew_grid(c, dn * modup_chunks(nl, c->K, chunk));
#define RF_MU(SC, CH)                                                                                            \
    hipLaunchKernelGGL((modup_bconv_kernel<SC, CH>), grid, dim3(kEw), 0, s, x, ext, c->d_pc, c->d_modup,          \
                       c->modup_stride, c->log_n, nl, c->L, c->K, c->alpha)
    if (scaled) {
        if (chunk == 4) RF_MU(true, 4);
        else if (chunk == 16) RF_MU(true, 16);
        else RF_MU(true, 8);
    } else {
        if (chunk == 4) RF_MU(false, 4);
        else if (chunk == 16) RF_MU(false, 16);
        else RF_MU(false, 8);
    }
#undef RF_MU
    return check_launch("modup_bconv");
}

template <int A, int B>
static void launch_ip(const rf_ctx *c, const uint64_t *d, const uint64_t *ext, const uint64_t *evk, uint64_t *ip,
                      uint32_t nl, hipStream_t s, const IpFold &f) {
    const dim3 grid(2 * c->K * (c->n / kMixTile) + nl * (c->n / kEw));
    if (c->fp_mask.any())
        hipLaunchKernelGGL((inner_product_kernel<A, B, FpMask>), grid, dim3(kEw), 0, s, d, ext, evk, ip, c->d_pc,
                           c->d_tw_inv, c->fp_mask, nl, c->L, c->K, c->alpha, f);
    else
        hipLaunchKernelGGL((inner_product_kernel<A, B, NoFp>), grid, dim3(kEw), 0, s, d, ext, evk, ip, c->d_pc,
                           c->d_tw_inv, NoFp{}, nl, c->L, c->K, c->alpha, f);
}

int launch_inner_product(const rf_ctx *c, const uint64_t *d, const uint64_t *ext, const uint64_t *evk, uint64_t *ip,
                         uint32_t nl, hipStream_t s, const IpFold &fold) {
    ProfScope prof("inner_product", s);
    IpFold f = fold;
    f.pinv = c->d_moddown + moddown_pinv_off(c);
    switch (c->log_n) {
        case 13: launch_ip<7, 6>(c, d, ext, evk, ip, nl, s, f); break;
        case 14: launch_ip<7, 7>(c, d, ext, evk, ip, nl, s, f); break;
        case 15: launch_ip<8, 7>(c, d, ext, evk, ip, nl, s, f); break;
        case 16: launch_ip<8, 8>(c, d, ext, evk, ip, nl, s, f); break;
        default: return fail(RF_EUNSUPPORTED, "inner product: ring degree");
    }
    return check_launch("inner_product");
}

int launch_automorphism(const rf_ctx *c, const uint64_t *in, uint64_t *out, uint32_t galois, uint32_t nl,
                        uint32_t n_polys, hipStream_t s) {
    ProfScope prof("automorphism", s);
    hipLaunchKernelGGL(automorphism_kernel, ew_grid(c, nl * n_polys), dim3(kEw), 0, s, in, out, galois, c->log_n);
    return check_launch("automorphism");
}

int launch_ewise(const rf_ctx *c, int op, const uint64_t *a, const uint64_t *b, int64_t k, uint64_t *out,
                 uint32_t nl, uint32_t n_polys, hipStream_t s) {
    ProfScope prof("elementwise", s);
    const dim3 g = ew_grid(c, nl * n_polys);
    switch (op) {
        case 0: hipLaunchKernelGGL(ewise_kernel<0>, g, dim3(kEw), 0, s, a, b, k, out, c->d_pc, c->log_n, nl); break;
        case 1: hipLaunchKernelGGL(ewise_kernel<1>, g, dim3(kEw), 0, s, a, b, k, out, c->d_pc, c->log_n, nl); break;
        case 2: hipLaunchKernelGGL(ewise_kernel<2>, g, dim3(kEw), 0, s, a, b, k, out, c->d_pc, c->log_n, nl); break;
        case 3: hipLaunchKernelGGL(ewise_kernel<3>, g, dim3(kEw), 0, s, a, b, k, out, c->d_pc, c->log_n, nl); break;
        case 4: hipLaunchKernelGGL(ewise_kernel<4>, g, dim3(kEw), 0, s, a, b, k, out, c->d_pc, c->log_n, nl); break;
        default: return fail(RF_EINVAL, "unknown element-wise op");
    }
    return check_launch("elementwise");
}

}  // namespace rf
