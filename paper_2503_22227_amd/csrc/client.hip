// Client side on the GPU: key generation, secret-key encryption, decryption,
// CRT composition and CKKS encode / decode (the create-key, encode, encrypt,
// decrypt and decode rows of the operator tables of section V-A; the client
// of the query framework, IV-A).  Random draws come in as arguments; the
// integer steps are exact, encode / decode run in double precision.
//
// Kernels are one thread per coefficient (grid.x over N in blocks of kCl,
// grid.y over limbs, grid.z over polynomials) except the FFT (four values per
// thread).
#include <hip/hip_runtime.h>

#include "ks_dev.hpp"
#include "ntt_dev.hpp"
#include "rf_internal.hpp"

namespace rf {

constexpr int kCl = 256;
constexpr int kCrtThreads = 128;

// Representative in [0, q) of a signed 64-bit integer.
__device__ __forceinline__ uint64_t signed_mod(int64_t v, const PrimeConst &pc) {
    const uint64_t mag = v < 0 ? (uint64_t)0 - (uint64_t)v : (uint64_t)v;
    const uint64_t r = barrett64(mag, pc.mu1, pc.mu0, pc.q);
    return (v < 0 && r) ? pc.q - r : r;
}

// Lift flags: the x term times floor(Q_L / t) (BFV message), the y term times t
// (BGV error), the x term times t (BGV key error).
enum LiftMode { kLiftXDelta = 1, kLiftYT = 2, kLiftXT = 4 };

// out[z][i][n] = x[z][n] (times the mode's factor) + y[z][n] (likewise) mod p_{first+i}.
__global__ __launch_bounds__(kCl) void lift_kernel(const int64_t *__restrict__ x, const int64_t *__restrict__ y,
                                                   size_t in_stride, uint64_t *__restrict__ out, size_t out_stride,
                                                   const PrimeConst *__restrict__ pcs, const uint64_t *__restrict__ cl,
                                                   uint32_t first, uint32_t log_n, int mode) {
    const uint32_t i = blockIdx.y, z = blockIdx.z, g = first + i;
    const size_t n = (size_t)blockIdx.x * kCl + threadIdx.x;
    const PrimeConst pc = pcs[g];
    uint64_t r = signed_mod(x[z * in_stride + n], pc);
    if (mode & kLiftXDelta) r = shoup(r, cl[4 * g + 2], cl[4 * g + 3], pc.q);
    if (mode & kLiftXT) r = shoup(r, pc.tmod, pc.tmod_p, pc.q);
    if (y) {
        uint64_t e = signed_mod(y[z * in_stride + n], pc);
        if (mode & kLiftYT) e = shoup(e, pc.tmod, pc.tmod_p, pc.q);
        r = addmod(r, e, pc.q);
    }
    out[z * out_stride + ((size_t)i << log_n) + n] = r;
}

// Encryption (CKKS, BGV) in the two passes of NTT(m + err e): the first lifts
// m + err e into the limb's prime, the last writes c0 = NTT(.) - a s and c1 = a.
// As launches of their own the lift, the product and the copy of a moved another
// 76 MB: 24 limbs at N = 2^16 took 55 us and the copy, now 40 us (HIP events).
struct EncryptPro {
    static constexpr bool kBlocked = false;
    const int64_t *m, *e;
    const PrimeConst *pc;
    bool err_t;  // BGV: err = t
    __device__ __forceinline__ uint64_t operator()(size_t n) const {
        uint64_t r = signed_mod(e[n], *pc);
        if (err_t) r = shoup(r, pc->tmod, pc->tmod_p, pc->q);
        return addmod(signed_mod(m[n], *pc), r, pc->q);
    }
    // any 64-bit integer, up to a multiple of q, below q + 2^32 in magnitude
    __device__ __forceinline__ static double lift(int64_t v, const FpMod &f) {
        return f.mul((double)(int32_t)(v >> 32), f.red(4294967296.0)) + (double)(uint32_t)v;
    }
    __device__ __forceinline__ double fp(size_t n, const FpMod &f) const {
        double r = lift(e[n], f);
        if (err_t) r = f.mul(r, f.centre(pc->tmod));
        return lift(m[n], f) + r;
    }
};

struct EncryptEpi {
    static constexpr bool kPrefetch = false, kBlocked = false;
    const uint64_t *a, *s;
    uint64_t *c0, *c1;
    uint64_t mu1, mu0, q;
    __device__ __forceinline__ void operator()(size_t n, uint64_t x) const {
        const uint64_t an = a[n];
        c0[n] = submod(x, mulmod(an, s[n], mu1, mu0, q), q);
        c1[n] = an;
    }
    __device__ __forceinline__ void fp(size_t n, double x, const FpMod &f) const {
        const uint64_t an = a[n];
        c0[n] = f.canon(f.red(x - f.mul(FpMod::from_u52(an), FpMod::from_u52(s[n]))));
        c1[n] = an;
    }
};

// Decryption (CKKS, BGV): c0 + c1 s as the prologue of the first pass of its INTT.
struct DecryptPro {
    static constexpr bool kBlocked = false;
    const uint64_t *c0, *c1, *s;
    uint64_t mu1, mu0, q;
    __device__ __forceinline__ uint64_t operator()(size_t n) const {
        return addmod(c0[n], mulmod(c1[n], s[n], mu1, mu0, q), q);
    }
    __device__ __forceinline__ double fp(size_t n, const FpMod &f) const {
        return FpMod::from_u52(c0[n]) + f.mul(FpMod::from_u52(c1[n]), FpMod::from_u52(s[n]));
    }
};

// PASS 0, 1: the two passes of an encryption; 2: the first of a decryption.
// TILE 4096 or, for launches with few limbs, 1024 (ntt_cols_small_pro).
struct ClientArgs {
    const int64_t *m, *e;
    const uint64_t *a, *s;  // encryption: the mask; decryption: the ciphertext; the secret
    uint64_t *out;
    const TwPair *tw;
    const PrimeConst *pcs;
    uint32_t nl;
    bool err_t;
};
constexpr int kClientE = 4;

template <int PASS, int A, int B, int TILE>
constexpr int client_waves() { return TILE == kTile ? ntt_waves(PASS == 0 ? A : B) : 2; }

template <int PASS, int A, int B, int TILE>
__global__ __launch_bounds__(TILE == kTile ? kThreads : TILE / kClientE)
    __attribute__((amdgpu_waves_per_eu(client_waves<PASS, A, B, TILE>()))) void client_pass_kernel(ClientArgs c, FpMask fpm) {
    constexpr int LOGN = A + B, S = PASS == 0 ? (1 << A) : (1 << B);
    __shared__ uint64_t lds[S * (TILE / S + 1)];
    const uint32_t i = blockIdx.y;
    const bool fp = fpm.has(i);
    const PrimeConst pc = c.pcs[i];
    const size_t li = (size_t)i << LOGN, poly = (size_t)c.nl << LOGN;
    const TwPair *tw = c.tw + li;
    uint64_t *out = c.out + li;
    if constexpr (PASS == 0) {
        const EncryptPro pro{c.m, c.e, c.pcs + i, c.err_t};
        if constexpr (TILE == kTile) ntt_cols_unit_pro<A, B, true>(lds, out, tw, pc, fp, blockIdx.x, pro);
        else ntt_cols_small_pro<A, B, true, TILE, kClientE>(lds, pro, out, tw, pc, fp, blockIdx.x);
    } else if constexpr (PASS == 1) {
        const EncryptEpi epi{c.a + li, c.s + li, out, out + poly, pc.mu1, pc.mu0, pc.q};
        if constexpr (TILE == kTile) ntt_rows_unit_epi<A, B>(lds, out, tw, pc, fp, blockIdx.x, epi);
        else ntt_rows_small_pe<A, B, true, TILE, kClientE>(lds, RawPro{out}, tw, pc, fp, blockIdx.x, epi);
    } else {
        const DecryptPro pro{c.a + li, c.a + poly + li, c.s + li, pc.mu1, pc.mu0, pc.q};
        if constexpr (TILE == kTile) ntt_rows_unit_pe<A, B, false>(lds, pro, tw, pc, fp, blockIdx.x, RawEpi{out});
        else ntt_rows_small_pe<A, B, false, TILE, kClientE>(lds, pro, tw, pc, fp, blockIdx.x, RawEpi{out});
    }
}

// SUB: out = x - a s; otherwise out = x + a s (limb i mod q_i, s limb i of [L+K][N]).
template <bool SUB>
__global__ __launch_bounds__(kCl) void fma_s_kernel(const uint64_t *x, const uint64_t *__restrict__ a,
                                                    const uint64_t *__restrict__ s, uint64_t *out,
                                                    const PrimeConst *__restrict__ pcs, uint32_t log_n) {
    const uint32_t i = blockIdx.y;
    const size_t off = ((size_t)i << log_n) + (size_t)blockIdx.x * kCl + threadIdx.x;
    const PrimeConst pc = pcs[i];
    const uint64_t as = mulmod(a[off], s[off], pc.mu1, pc.mu0, pc.q);
    out[off] = SUB ? submod(x[off], as, pc.q) : addmod(x[off], as, pc.q);
}

// Switching-key assembly of digit j = blockIdx.z on limb m = blockIdx.y of Q_L u P:
// evk[j][0][m] (holding NTT(err e_j) on entry) += -a_j s + [m in D_j] [P]_{q_m} s',
// s' = s^2 (galois 0) or sigma_g(s); evk[j][1][m] = a_j.
__global__ __launch_bounds__(kCl) void keygen_kernel(uint64_t *evk, const uint64_t *__restrict__ a,
                                                     const uint64_t *__restrict__ s, const PrimeConst *__restrict__ pcs,
                                                     const uint64_t *__restrict__ cl, uint32_t galois, uint32_t log_n,
                                                     uint32_t L, uint32_t K, uint32_t alpha) {
    const uint32_t m = blockIdx.y, j = blockIdx.z;
    const uint32_t n = blockIdx.x * kCl + threadIdx.x;
    const size_t limbs = (size_t)(L + K) << log_n;
    const size_t off = ((size_t)m << log_n) + n;
    const PrimeConst pc = pcs[m];
    uint64_t *b = evk + 2 * (size_t)j * limbs;
    const uint64_t aj = a[(size_t)j * limbs + off];
    const uint64_t sm = s[off];
    uint64_t v = submod(b[off], mulmod(aj, sm, pc.mu1, pc.mu0, pc.q), pc.q);
    if (m < L && m >= j * alpha && m < j * alpha + alpha) {
        const uint64_t sf = galois ? s[((size_t)m << log_n) + galois_src(n, galois, log_n)]
                                   : mulmod(sm, sm, pc.mu1, pc.mu0, pc.q);
        v = addmod(v, shoup(sf, cl[4 * m], cl[4 * m + 1], pc.q), pc.q);
    }
    b[off] = v;
    b[limbs + off] = aj;
}

// Balanced mixed-radix digits of each coefficient, X = sum_i v_i q_0 .. q_{i-1}
// with v_i in (-q_i/2, q_i/2]: a complete residue system, so X is the centred
// representative mod Q_l.  Horner in double from the top digit, then / scale.
__global__ __launch_bounds__(kCrtThreads) void crt_centered_kernel(const uint64_t *__restrict__ x, double *out,
                                                                   const PrimeConst *__restrict__ pcs,
                                                                   const uint64_t *__restrict__ gar, uint32_t L,
                                                                   uint32_t nl, uint32_t log_n, double scale) {
    __shared__ int64_t v[kMaxCrtLimbs][kCrtThreads];
    const size_t n = (size_t)blockIdx.x * kCrtThreads + threadIdx.x;
    const int tid = threadIdx.x;
    for (uint32_t j = 0; j < nl; ++j) {
        const PrimeConst pc = pcs[j];
        uint64_t t = x[((size_t)j << log_n) + n];
        for (uint32_t i = 0; i < j; ++i) {
            const uint64_t *gi = gar + ((size_t)i * L + j) * 2;
            t = shoup(submod(t, signed_mod(v[i][tid], pc), pc.q), gi[0], gi[1], pc.q);
        }
        v[j][tid] = t > (pc.q >> 1) ? (int64_t)t - (int64_t)pc.q : (int64_t)t;
    }
    double acc = (double)v[nl - 1][tid];
    for (int i = (int)nl - 2; i >= 0; --i) acc = fma(acc, (double)pcs[i].q, (double)v[i][tid]);
    out[n] = acc / scale;
}

// The same digits where every limb but the first is below kFpPrimeBound, in FP64
// (FpMod).  A step takes the next digit v = v_i and updates every limb above it,
// t_j <- (t_j - v) q_i^-1 mod q_j, so the updates of one step do not wait for
// each other (the kernel above runs one chain of nl^2 / 2 dependent products per
// coefficient).  The limbs move down one register a step, which keeps the register
// indices fixed while the loop over the steps stays rolled; W is the width of the
// last 8, 16, 24 or 32 limbs.  Bound by FP64 latency with one wave per SIMD at N =
// 2^16: 17 limbs 51.1 us by the kernel above, 24.4 us here (HIP events); 27.5 us
// before the constants of a step were contiguous.
template <int W>
__device__ __forceinline__ void crt_steps(double (&t)[32], uint32_t &i, uint32_t nl, double *v_out, double &v,
                                          const double2 *__restrict__ qq, const double *__restrict__ gar,
                                          uint32_t stride) {
#pragma unroll 1
    for (; i < nl && nl - i > (uint32_t)W - 8; ++i) {
        // t[k] is limb i + k, short of v_{i-1}: its step, then digit i
        // (the tables are padded: the registers past the last limb hold nothing)
        const double *gi = gar + (size_t)(i - 1) * stride + i;
#pragma unroll
        for (int k = 0; k < W; ++k) {
            const FpMod f{qq[i + k].x, qq[i + k].y};
            t[k] = f.mul(t[k] - v, gi[k]);
        }
        const FpMod f{qq[i].x, qq[i].y};
        v = f.red(t[0]);
        const double half = 0.5 * f.q;
        v = v > half ? v - f.q : (v < -half ? v + f.q : v);
        v_out[(size_t)i * kCrtThreads] = v;
#pragma unroll
        for (int k = 0; k + 1 < W; ++k) t[k] = t[k + 1];
    }
}

__global__ __launch_bounds__(kCrtThreads) void crt_centered_narrow_kernel(const uint64_t *__restrict__ x, double *out,
                                                                          const PrimeConst *__restrict__ pcs,
                                                                          const double *__restrict__ gar, uint32_t L,
                                                                          uint32_t nl, uint32_t log_n, double scale,
                                                                          bool narrow0) {
    const uint32_t stride = L + kMaxCrtLimbs;
    const double2 *qq = (const double2 *)gar;  // (q_j, 1 / q_j), then the inverses
    gar += 2 * (size_t)stride;
    __shared__ double vs[kMaxCrtLimbs][kCrtThreads];
    const size_t n = (size_t)blockIdx.x * kCrtThreads + threadIdx.x;
    const int tid = threadIdx.x;
    double t[32];
    // limbs 1.. (limb 1 + k in t[k])
#pragma unroll
    for (int k = 0; k < 31; ++k) t[k] = 1 + k < (int)nl ? FpMod::from_u52(x[((size_t)(1 + k) << log_n) + n]) : 0.0;
    t[31] = 0.0;
    const uint64_t x0 = x[n], q0 = pcs[0].q;
    const int64_t v0 = x0 > (q0 >> 1) ? (int64_t)x0 - (int64_t)q0 : (int64_t)x0;
    vs[0][tid] = (double)v0;
    double v = (double)v0;
    if (!narrow0) {
        // a wide first digit: its residue mod every other prime, from its halves
        const double h = (double)(v0 >> 30), l = (double)(v0 & 0x3fffffff);
#pragma unroll
        for (int k = 0; k < 31; ++k) {
            if (1 + k < (int)nl) {
                const FpMod f{pcs[1 + k].qd, pcs[1 + k].qinv};
                t[k] -= f.mul(h, f.red(1073741824.0)) + l;
            }
        }
        v = 0.0;
    }
    uint32_t i = 1;
    crt_steps<32>(t, i, nl, &vs[0][tid], v, qq, gar, stride);
    crt_steps<24>(t, i, nl, &vs[0][tid], v, qq, gar, stride);
    crt_steps<16>(t, i, nl, &vs[0][tid], v, qq, gar, stride);
    crt_steps<8>(t, i, nl, &vs[0][tid], v, qq, gar, stride);
    double acc = vs[nl - 1][tid];
    for (int k = (int)nl - 2; k >= 0; --k) acc = fma(acc, (double)pcs[k].q, vs[k][tid]);
    out[n] = acc / scale;
}

// FFT of N = 2^(LA + LB) complex values in two launches.  It is the radix-2
// decimation in time over the points x[q + (N / S) m] (log2 N stages, stage Ns
// combining two sub-transforms of Ns points with the twiddles
// exp(sign 2 pi i k / (2 Ns)) = zeta^(+-k N / Ns)): the first launch runs the
// stages up to 2^LA points, for which it needs 2^LA points N / 2^LA apart, the
// second the rest, for which it needs the points with one k mod 2^LA.  A
// workgroup holds 1024 values, U = 1024 / S neighbouring sub-transforms of S
// points, 4 per thread: two stages at a time in registers, exchanged through two
// LDS buffers.  All twiddles of a thread are fetched together with its values.
// One launch per stage took 40 us at N = 2^16 and the steps before and after 13 us,
// latency all of it; the two launches take 14 us (HIP events).
constexpr int kFftThreads = 256, kFftTile = 1024;

__device__ __forceinline__ double2 fft_twiddle(const double2 *__restrict__ zeta, uint32_t k, uint32_t log_n,
                                               uint32_t log_ns, int sign) {
    const uint32_t two_n = 2u << log_n;
    uint32_t e = k << (log_n - log_ns);
    if (sign < 0) e = (two_n - e) & (two_n - 1);
    return zeta[e];
}

// (a, b) <- (a + b w, a - b w), the products rounded as written here: encoded
// coefficients are whole numbers, so the rounding is part of the result.
__device__ __forceinline__ void fft_bfly(double2 &a, double2 &b, const double2 &w) {
#pragma clang fp contract(off)
    const double2 v1 = make_double2(__builtin_fma(b.x, w.x, -(b.y * w.y)), __builtin_fma(b.y, w.x, b.x * w.y));
    b = make_double2(a.x - v1.x, a.y - v1.y);
    a = make_double2(a.x + v1.x, a.y + v1.y);
}

// Stages of 2^LS points: in(p) the p-th value of this thread's sub-transform u
// (p = j + c S / 4 in turn), out(p, value) its results.  k0 + (k << LK): the
// index that sets the twiddles (k0 < 2^LK from the stages before).
template <int LS, int LK, typename In, typename Out>
__device__ __forceinline__ void fft_stages(double2 (*lds)[kFftTile], const double2 *__restrict__ zeta, uint32_t log_n,
                                           int sign, uint32_t k0, const In &in, const Out &out) {
    constexpr int S = 1 << LS, U = kFftTile / S, Q = S / 4, R4 = LS / 2;
    const int u = threadIdx.x % U, j = threadIdx.x / U;  // j < Q
    double2 v[4], w[R4][3], wl[2];
#pragma unroll
    for (int c = 0; c < 4; ++c) v[c] = in(j + c * Q);
#pragma unroll
    for (int r = 0; r < R4; ++r) {
        const uint32_t ns = 1u << (2 * r), k = (uint32_t)j & (ns - 1);
        w[r][0] = fft_twiddle(zeta, k0 + (k << LK), log_n, LK + 2 * r, sign);
        w[r][1] = fft_twiddle(zeta, k0 + (k << LK), log_n, LK + 2 * r + 1, sign);
        w[r][2] = fft_twiddle(zeta, k0 + ((k + ns) << LK), log_n, LK + 2 * r + 1, sign);
    }
    if constexpr (LS & 1) {
        // the last stage alone: butterflies (j, j + S / 2) and (j + Q, j + Q + S / 2)
#pragma unroll
        for (int c = 0; c < 2; ++c)
            wl[c] = fft_twiddle(zeta, k0 + ((uint32_t)(j + c * Q) << LK), log_n, LK + LS - 1, sign);
    }
#pragma unroll
    for (int r = 0; r < R4; ++r) {
        const int ns = 1 << (2 * r), k = j & (ns - 1), q = j >> (2 * r);
        fft_bfly(v[0], v[2], w[r][0]);
        fft_bfly(v[1], v[3], w[r][0]);
        // (v0, v2) = k, k + ns of group q; (v1, v3) the same of group q + Q / ns
        fft_bfly(v[0], v[1], w[r][1]);
        fft_bfly(v[2], v[3], w[r][2]);
        const int d = q * 4 * ns + k;
        if (!(LS & 1) && r == R4 - 1) {
            out(d, v[0]);
            out(d + ns, v[2]);
            out(d + 2 * ns, v[1]);
            out(d + 3 * ns, v[3]);
        } else {
            double2 *b = lds[r & 1];
            b[d * U + u] = v[0];
            b[(d + ns) * U + u] = v[2];
            b[(d + 2 * ns) * U + u] = v[1];
            b[(d + 3 * ns) * U + u] = v[3];
            __syncthreads();
#pragma unroll
            for (int c = 0; c < 4; ++c) v[c] = b[(j + c * Q) * U + u];
        }
    }
    if constexpr (LS & 1) {
        fft_bfly(v[0], v[2], wl[0]);
        fft_bfly(v[1], v[3], wl[1]);
        out(j, v[0]);
        out(j + S / 2, v[2]);
        out(j + Q, v[1]);
        out(j + Q + S / 2, v[3]);
    }
}

// First launch.  Decode: the values are y_i = x_i zeta^i (the negacyclic twist).
// Encode: the value at zeta^(2t+1) for every t, z_j at 2t+1 = 5^j mod 2N and its
// conjugate at 2N - 5^j (t' = N - 1 - t); slot_of[t] = j, or j | 2^31 for the
// conjugate.
template <int LA, int LB, bool DECODE>
__global__ __launch_bounds__(kFftThreads) void fft_first_kernel(const double *__restrict__ src, double2 *__restrict__ mid,
                                                                const double2 *__restrict__ zeta,
                                                                const uint32_t *__restrict__ slot_of) {
    __shared__ double2 lds[2][kFftTile];
    constexpr int LN = LA + LB, U = kFftTile >> LA;
    const uint32_t q = blockIdx.x * U + threadIdx.x % U;
    auto in = [&](int m) -> double2 {
        const uint32_t i = q + ((uint32_t)m << LB);
        if constexpr (DECODE) {
            const double2 w = zeta[i];
            const double x = src[i];
            return make_double2(x * w.x, x * w.y);
        } else {
            const uint32_t j = slot_of[i];
            const double2 z = ((const double2 *)src)[j & 0x7fffffffu];
            return make_double2(z.x, (j >> 31) ? -z.y : z.y);
        }
    };
    auto out = [&](int k, const double2 &v) { mid[((size_t)q << LA) + k] = v; };
    fft_stages<LA, 0>(lds, zeta, LN, DECODE ? 1 : -1, 0, in, out);
}

// Second launch.  Decode: slot j is the value at t = (5^j mod 2N - 1) / 2.
// Encode: m_i = round(Re(zeta^-i U_i) factor), clamped to |m| <= 2^62.
template <int LA, int LB, bool DECODE>
__global__ __launch_bounds__(kFftThreads) void fft_second_kernel(const double2 *__restrict__ mid, void *__restrict__ dst,
                                                                 const double2 *__restrict__ zeta,
                                                                 const uint32_t *__restrict__ slot_of, double factor) {
    __shared__ double2 lds[2][kFftTile];
    constexpr int LN = LA + LB, U = kFftTile >> LB;
    constexpr uint32_t N = 1u << LN;
    const uint32_t k0 = blockIdx.x * U + threadIdx.x % U;
    auto in = [&](int q) -> double2 { return mid[((size_t)q << LA) + k0]; };
    auto out = [&](int k1, const double2 &v) {
        const uint32_t i = k0 + ((uint32_t)k1 << LA);
        if constexpr (DECODE) {
            const uint32_t j = slot_of[i];
            if (!(j >> 31)) ((double2 *)dst)[j] = v;
        } else {
            const double2 w = zeta[(2 * N - i) & (2 * N - 1)];
            double re = rint(__builtin_fma(w.x, v.x, -(w.y * v.y)) * factor);
            const double lim = 4611686018427387904.0;  // 2^62
            re = fmin(fmax(re, -lim), lim);
            ((int64_t *)dst)[i] = (int64_t)re;
        }
    };
    fft_stages<LB, LA>(lds, zeta, LN, DECODE ? 1 : -1, k0, in, out);
}

}  // namespace rf

using namespace rf;

namespace {

bool overlaps_bytes(const void *a, size_t na, const void *b, size_t nb) {
    const char *x = (const char *)a, *y = (const char *)b;
    return x < y + nb && y < x + na;
}

int check_launch(const char *what) {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(RF_EHIP, std::string(what) + ": " + hipGetErrorString(e));
    return RF_OK;
}

struct Dev {
    int prev = -1;
    explicit Dev(int d) {
        if (hipGetDevice(&prev) != hipSuccess) prev = -1;
        if (prev != d) (void)hipSetDevice(d);
    }
    ~Dev() {
        int cur = -1;
        if (prev >= 0 && hipGetDevice(&cur) == hipSuccess && cur != prev) (void)hipSetDevice(prev);
    }
};

NttBatch plain_batch(const rf_ctx *c, uint64_t *d, uint64_t stride, uint32_t per_poly, uint32_t n_polys) {
    NttBatch b;
    b.in = d;
    b.out = d;
    b.in_poly_stride = stride;
    b.out_poly_stride = stride;
    b.per_poly = per_poly;
    b.n_polys = n_polys;
    b.prime_base = 0;
    b.pmap = nullptr;
    b.order = c->order(per_poly <= c->L ? c->q_order[per_poly] : c->all_order);
    return b;
}

int lift(const rf_ctx *c, const int64_t *x, const int64_t *y, size_t in_stride, uint64_t *out, size_t out_stride,
         uint32_t first, uint32_t nlimbs, uint32_t npolys, int mode, hipStream_t s) {
    ProfScope prof("client_lift", s);
    hipLaunchKernelGGL(lift_kernel, dim3(c->n / kCl, nlimbs, npolys), dim3(kCl), 0, s, x, y, in_stride, out,
                       out_stride, c->d_pc, c->d_client, first, c->log_n, mode);
    return check_launch("lift");
}

// One of the client's transform passes over nl limbs, two-pass ring degrees.
template <int PASS>
int client_pass(const rf_ctx *c, ClientArgs a, hipStream_t s, const char *name) {
    // small tiles while 4096-residue ones would leave CUs idle (as the NTT's default)
    const bool small = a.nl * (c->n / kTile) < kDefaultTuning.ntt_small_below;
    const TwPair *rows = PASS == 1 ? (small ? c->d_tw_fwd : c->d_tw_fwd_rows) : (small ? c->d_tw_inv : c->d_tw_inv_rows);
    a.tw = PASS == 0 ? c->d_tw_fwd : rows;
    a.pcs = c->d_pc;
    ProfScope prof(name, s);
#define RF_CP(A, B)                                                                                              \
    if (small)                                                                                                   \
        hipLaunchKernelGGL((client_pass_kernel<PASS, A, B, 1024>), dim3(c->n / 1024, a.nl), dim3(1024 / kClientE), \
                           0, s, a, c->fp_mask);                                                                 \
    else                                                                                                         \
        hipLaunchKernelGGL((client_pass_kernel<PASS, A, B, kTile>), dim3(c->n / kTile, a.nl), dim3(kThreads), 0,  \
                           s, a, c->fp_mask)
    switch (c->log_n) {
        case 13: RF_CP(7, 6); break;
        case 14: RF_CP(7, 7); break;
        case 15: RF_CP(8, 7); break;
        case 16: RF_CP(8, 8); break;
        default: return fail(RF_EUNSUPPORTED, "client pass: ring degree");
    }
#undef RF_CP
    return check_launch(name);
}

template <bool DECODE>
int fft(const rf_ctx *c, const double *src, double2 *mid, void *dst, double factor, hipStream_t s) {
    const dim3 g(c->n / kFftTile), b(kFftThreads);
    const double2 *zeta = (const double2 *)c->d_zeta;
#define RF_FFT(LA, LB)                                                                                           \
    {                                                                                                            \
        {                                                                                                        \
            ProfScope prof("client_fft", s);                                                                     \
            hipLaunchKernelGGL((fft_first_kernel<LA, LB, DECODE>), g, b, 0, s, src, mid, zeta, c->d_slot_of);     \
        }                                                                                                        \
        ProfScope prof("client_fft", s);                                                                         \
        hipLaunchKernelGGL((fft_second_kernel<LA, LB, DECODE>), g, b, 0, s, mid, dst, zeta, c->d_slot_of, factor); \
    }
    switch (c->log_n) {
        case 12: RF_FFT(6, 6) break;
        case 13: RF_FFT(7, 6) break;
        case 14: RF_FFT(7, 7) break;
        case 15: RF_FFT(8, 7) break;
        case 16: RF_FFT(8, 8) break;
        default: return fail(RF_EUNSUPPORTED, "FFT: ring degree");
    }
#undef RF_FFT
    return check_launch(DECODE ? "decode" : "encode");
}

}  // namespace

extern "C" int rf_key_ntt(const rf_ctx *c, const int64_t *x, uint64_t *out, void *stream) {
    if (!c || !x || !out) return fail(RF_EINVAL, "rf_key_ntt: null argument");
    Dev g(c->device);
    hipStream_t s = (hipStream_t)stream;
    const uint32_t all = c->L + c->K;
    int rc;
    if ((rc = lift(c, x, nullptr, 0, out, 0, 0, all, 1, 0, s))) return rc;
    return launch_ntt(c, plain_batch(c, out, 0, all, 1), true, s);
}

extern "C" int rf_keygen_switch(const rf_ctx *c, const uint64_t *s_ntt, uint32_t galois, const uint64_t *a,
                                const int64_t *e, uint64_t *evk, void *stream) {
    if (!c || !s_ntt || !a || !e || !evk) return fail(RF_EINVAL, "rf_keygen_switch: null argument");
    if (galois != 0 && ((galois & 1u) == 0 || galois >= 2u * c->n))
        return fail(RF_EINVAL, "rf_keygen_switch: Galois element must be 0 (relinearisation) or odd and < 2N");
    const uint32_t all = c->L + c->K;
    const size_t limbs = (size_t)all * c->n;
    const size_t key_bytes = (size_t)c->dnum * 2 * limbs * 8;
    if (overlaps_bytes(evk, key_bytes, s_ntt, limbs * 8) || overlaps_bytes(evk, key_bytes, a, c->dnum * limbs * 8))
        return fail(RF_EINVAL, "rf_keygen_switch: evk overlaps an input");
    Dev g(c->device);
    hipStream_t s = (hipStream_t)stream;
    int rc;
    // NTT(err e_j) into polynomial 0 of every digit
    if ((rc = lift(c, e, nullptr, c->n, evk, 2 * limbs, 0, all, c->dnum, c->scheme == RF_BGV ? kLiftXT : 0, s)))
        return rc;
    if ((rc = launch_ntt(c, plain_batch(c, evk, 2 * limbs, all, c->dnum), true, s))) return rc;
    {
        ProfScope prof("client_keygen", s);
        hipLaunchKernelGGL(keygen_kernel, dim3(c->n / kCl, all, c->dnum), dim3(kCl), 0, s, evk, a, s_ntt, c->d_pc,
                           c->d_client, galois, c->log_n, c->L, c->K, c->alpha);
    }
    return check_launch("keygen");
}

extern "C" int rf_encrypt_sk(const rf_ctx *c, const int64_t *m, const int64_t *e, const uint64_t *a,
                             const uint64_t *s_ntt, uint64_t *out, uint32_t nl, void *stream) {
    if (!c || !m || !e || !a || !s_ntt || !out) return fail(RF_EINVAL, "rf_encrypt_sk: null argument");
    if (nl < 1 || nl > c->L) return fail(RF_ELEVEL, "rf_encrypt_sk: limb count out of range");
    if (c->scheme == RF_BFV && nl != c->L) return fail(RF_ELEVEL, "rf_encrypt_sk: BFV ciphertexts carry all L limbs");
    const size_t poly = (size_t)nl * c->n;
    if (overlaps_bytes(out, 2 * poly * 8, a, poly * 8) ||
        overlaps_bytes(out, 2 * poly * 8, s_ntt, (size_t)(c->L + c->K) * c->n * 8) ||
        overlaps_bytes(out, 2 * poly * 8, m, c->n * 8) || overlaps_bytes(out, 2 * poly * 8, e, c->n * 8))
        return fail(RF_EINVAL, "rf_encrypt_sk: out overlaps an input");
    Dev g(c->device);
    hipStream_t s = (hipStream_t)stream;
    uint64_t *c0 = out, *c1 = out + poly;
    int rc;
    if (c->scheme == RF_BFV) {
        // c1 <- Delta m + e; c0 <- INTT(NTT(a) s); c0 <- c1 - c0; c1 <- a
        if ((rc = lift(c, m, e, 0, c1, 0, 0, nl, 1, kLiftXDelta, s))) return rc;
        if (hipMemcpyAsync(c0, a, poly * 8, hipMemcpyDeviceToDevice, s) != hipSuccess)
            return fail(RF_EHIP, "rf_encrypt_sk: copy");
        if ((rc = launch_ntt(c, plain_batch(c, c0, 0, nl, 1), true, s))) return rc;
        if ((rc = launch_ewise(c, 4, c0, s_ntt, 0, c0, nl, 1, s))) return rc;
        if ((rc = launch_ntt(c, plain_batch(c, c0, 0, nl, 1), false, s))) return rc;
        if ((rc = launch_ewise(c, 1, c1, c0, 0, c0, nl, 1, s))) return rc;
    } else if (c->log_n > 12) {
        // (NTT(m + err e) - a s, a) in the transform's two passes
        ClientArgs ca{m, e, a, s_ntt, c0, nullptr, nullptr, nl, c->scheme == RF_BGV};
        if ((rc = client_pass<0>(c, ca, s, "client_encrypt_cols"))) return rc;
        return client_pass<1>(c, ca, s, "client_encrypt_rows");
    } else {
        // c0 <- NTT(m + err e) - a s
        if ((rc = lift(c, m, e, 0, c0, 0, 0, nl, 1, c->scheme == RF_BGV ? kLiftYT : 0, s))) return rc;
        if ((rc = launch_ntt(c, plain_batch(c, c0, 0, nl, 1), true, s))) return rc;
        {
            ProfScope prof("client_encrypt", s);
            hipLaunchKernelGGL(fma_s_kernel<true>, dim3(c->n / kCl, nl), dim3(kCl), 0, s, c0, a, s_ntt, c0, c->d_pc,
                               c->log_n);
        }
        if ((rc = check_launch("encrypt"))) return rc;
    }
    if (hipMemcpyAsync(c1, a, poly * 8, hipMemcpyDeviceToDevice, s) != hipSuccess)
        return fail(RF_EHIP, "rf_encrypt_sk: copy");
    return RF_OK;
}

extern "C" int rf_decrypt(const rf_ctx *c, const uint64_t *ct, const uint64_t *s_ntt, uint64_t *out, uint32_t nl,
                          void *stream) {
    if (!c || !ct || !s_ntt || !out) return fail(RF_EINVAL, "rf_decrypt: null argument");
    if (nl < 1 || nl > c->L) return fail(RF_ELEVEL, "rf_decrypt: limb count out of range");
    if (c->scheme == RF_BFV && nl != c->L) return fail(RF_ELEVEL, "rf_decrypt: BFV ciphertexts carry all L limbs");
    const size_t poly = (size_t)nl * c->n;
    if (overlaps_bytes(out, poly * 8, ct, 2 * poly * 8)) return fail(RF_EINVAL, "rf_decrypt: out overlaps ct");
    Dev g(c->device);
    hipStream_t s = (hipStream_t)stream;
    int rc;
    if (c->scheme == RF_BFV) {
        // c0 + INTT(NTT(c1) s)
        if (hipMemcpyAsync(out, ct + poly, poly * 8, hipMemcpyDeviceToDevice, s) != hipSuccess)
            return fail(RF_EHIP, "rf_decrypt: copy");
        if ((rc = launch_ntt(c, plain_batch(c, out, 0, nl, 1), true, s))) return rc;
        if ((rc = launch_ewise(c, 4, out, s_ntt, 0, out, nl, 1, s))) return rc;
        if ((rc = launch_ntt(c, plain_batch(c, out, 0, nl, 1), false, s))) return rc;
        return launch_ewise(c, 0, out, ct, 0, out, nl, 1, s);
    }
    if (c->log_n > 12) {
        // c0 + c1 s in the first pass of its INTT
        ClientArgs ca{nullptr, nullptr, ct, s_ntt, out, nullptr, nullptr, nl, false};
        if ((rc = client_pass<2>(c, ca, s, "client_decrypt_rows"))) return rc;
        return launch_intt_cols(c, plain_batch(c, out, 0, nl, 1), s);
    }
    {
        ProfScope prof("client_decrypt", s);
        hipLaunchKernelGGL(fma_s_kernel<false>, dim3(c->n / kCl, nl), dim3(kCl), 0, s, ct, ct + poly, s_ntt, out,
                           c->d_pc, c->log_n);
    }
    if ((rc = check_launch("decrypt"))) return rc;
    return launch_ntt(c, plain_batch(c, out, 0, nl, 1), false, s);
}

extern "C" int rf_crt_centered(const rf_ctx *c, const uint64_t *x, double *out, uint32_t nl, double scale,
                               void *stream) {
    if (!c || !x || !out) return fail(RF_EINVAL, "rf_crt_centered: null argument");
    if (nl < 1 || nl > c->L) return fail(RF_ELEVEL, "rf_crt_centered: limb count out of range");
    if (nl > kMaxCrtLimbs) return fail(RF_EUNSUPPORTED, "rf_crt_centered: at most 32 limbs");
    if (!(scale > 0.0)) return fail(RF_EINVAL, "rf_crt_centered: scale must be positive");
    if (overlaps_bytes(out, (size_t)c->n * 8, x, (size_t)nl * c->n * 8))
        return fail(RF_EINVAL, "rf_crt_centered: out overlaps x");
    Dev g(c->device);
    hipStream_t s = (hipStream_t)stream;
    {
        // the limbs after the first below the FP64 bound: a 60-bit prime may lead the chain
        bool narrow = true;
        for (uint32_t i = 1; i < nl; ++i) narrow = narrow && c->fp_mask.has(i);
        ProfScope prof("client_crt", s);
        if (narrow)
            hipLaunchKernelGGL(crt_centered_narrow_kernel, dim3(c->n / kCrtThreads), dim3(kCrtThreads), 0, s, x, out,
                               c->d_pc, c->d_garner_fp, c->L, nl, c->log_n, scale, c->fp_mask.has(0));
        else
            hipLaunchKernelGGL(crt_centered_kernel, dim3(c->n / kCrtThreads), dim3(kCrtThreads), 0, s, x, out, c->d_pc,
                               c->d_garner, c->L, nl, c->log_n, scale);
    }
    return check_launch("crt_centered");
}

extern "C" int rf_encode_ckks(const rf_ctx *c, const double *z, double scale, int64_t *m, void *ws, size_t ws_bytes,
                              void *stream) {
    if (!c || !z || !m) return fail(RF_EINVAL, "rf_encode_ckks: null argument");
    if (c->scheme != RF_CKKS) return fail(RF_EUNSUPPORTED, "rf_encode_ckks: CKKS contexts only");
    if (!(scale > 0.0)) return fail(RF_EINVAL, "rf_encode_ckks: scale must be positive");
    const size_t need = rf_workspace_bytes(c, RF_OP_ENCODE, 1);
    if (!ws || ws_bytes < need) return fail(RF_EWORKSPACE, "rf_encode_ckks: workspace too small");
    Dev g(c->device);
    hipStream_t s = (hipStream_t)stream;
    return fft<false>(c, z, (double2 *)ws, m, scale / (double)c->n, s);
}

extern "C" int rf_decode_ckks(const rf_ctx *c, const double *x, double *z, void *ws, size_t ws_bytes, void *stream) {
    if (!c || !x || !z) return fail(RF_EINVAL, "rf_decode_ckks: null argument");
    if (c->scheme != RF_CKKS) return fail(RF_EUNSUPPORTED, "rf_decode_ckks: CKKS contexts only");
    const size_t need = rf_workspace_bytes(c, RF_OP_DECODE, 1);
    if (!ws || ws_bytes < need) return fail(RF_EWORKSPACE, "rf_decode_ckks: workspace too small");
    Dev g(c->device);
    hipStream_t s = (hipStream_t)stream;
    return fft<true>(c, x, (double2 *)ws, z, 0.0, s);
}
